// Exercises the launch planner of the attention calls (host arithmetic, paper_2502_02534_amd/csrc/plan.h)
// under AddressSanitizer and UndefinedBehaviorSanitizer over a grid of descriptions and bounds, and
// checks the invariants the kernels rely on.  Exit status 0 = nothing found.
#include "../../paper_2502_02534_amd/csrc/plan.h"

#include <cstdio>
#include <initializer_list>
#include <vector>

using namespace spd::plan;

static int fail(const char* what, long long a, long long b)
{
    std::printf("FAILED: %s (%lld, %lld)\n", what, a, b);
    return 1;
}

// Order of the suffix items: every (sample, chunk) once, and a sample's chunks on at least half of the eight XCDs (four
// wavefront items a workgroup, workgroups to the XCDs in turn).
static int check_suffix_order()
{
    for (unsigned heads : {4u, 8u, 16u, 32u})
        for (unsigned samples = 1; samples <= 132; ++samples) {
            const unsigned chunks = 8;
            std::vector<char> seen(samples * chunks, 0);
            std::vector<unsigned> xcds(samples, 0u);
            for (unsigned unit = 0; unit < samples * chunks; ++unit) {
                const SuffixPlace at = suffix_place(unit, samples);
                if (at.n < 0 || at.n >= (int)samples || at.chunk < 0 || at.chunk >= (int)chunks || seen[at.n * chunks + at.chunk]++)
                    return fail("suffix order is no permutation", samples, unit);
                for (unsigned head = 0; head < heads; ++head)
                    xcds[at.n] |= 1u << ((unit * heads + head) / 4 % 8);
            }
            for (unsigned n = 0; n < samples; ++n)
                if (__builtin_popcount(xcds[n]) < 4)
                    return fail("a sample's chunks are on too few XCDs", samples, heads);
        }
    return 0;
}

// Where the suffix pass does not share the prefix pass's launch (32 query heads per KV head, too many groups), the prefix
// pass gets a workgroup per CU whatever the suffixes are.
static int check_two_launches()
{
    for (int hq : {16, 32})
        for (int groups : {1, 70000}) {
            const int n = groups > 1 ? groups : 256;
            spd_attn_desc d = {SPD_BF16, hq, 1, 128, groups, n, groups > 1 ? 1 : 256, 0, 0.f, 0};
            Plan with, without;
            if (make_plan(&d, 1024, 2048, &with) != SPD_OK || make_plan(&d, 1024, 0, &without) != SPD_OK)
                return fail("make_plan refused a valid description", hq, groups);
            const bool one = hq == 16 && groups == 1;
            if (one_launch(&d, groups) != one || (!one && with.prefix_split_tokens != without.prefix_split_tokens) ||
                (!one && with.fold_tokens != 0.0) || (one && with.prefix_split_tokens <= without.prefix_split_tokens))
                return fail("prefix plan of two launches", hq, with.prefix_split_tokens);
        }
    return 0;
}

// What of the suffix KV is marked as streamed, on both sides of the lines (bytes by the bounds of 8 KV heads of 128
// bf16 channels: 4096 a token), in whole calls and in trees.
static int check_stream()
{
    const long long v_line = 192ll * 1024 * 1024 / 4096, k_line = 1024ll * 1024 * 1024 / 4096;
    for (int page : {0, 16})
        for (int prefix : {0, 1000})
            for (int side = 0; side < 2; ++side)
                for (int levels : {1, 3}) {
                    spd_prefix_level lv[3] = {};
                    for (int l = 0; l < levels; ++l) {
                        lv[l].num_groups = l + 1;
                        lv[l].max_len = prefix;
                    }
                    const long long before = levels == 1 ? prefix : 6ll * prefix;
                    spd_attn_desc d = {SPD_BF16, 32, 8, 128, 1, 1, 0, page, 0.f, 0};
                    if (plan_stream(&d, levels, lv, v_line - before - 1 + side) != side)
                        return fail("line of the streamed V", before, side);
                    if (plan_stream(&d, levels, lv, k_line - before - 1 + side) != (side && !page ? 2 : 1))
                        return fail("line of the streamed K", before, side);
                }
    // 32 samples x 8 KV heads of up to 512 tokens after a 16k prompt, 128 MiB: kept
    spd_attn_desc d = {SPD_BF16, 64, 8, 128, 1, 32, 32, 0, 0.f, 0};
    spd_prefix_level lv = {};
    lv.num_groups = 1;
    lv.max_len = 16384;
    if (plan_stream(&d, 1, &lv, 512) != 0)
        return fail("a call of half the cache is streamed", 0, 0);
    return 0;
}

// General kernel: one workgroup per CU and no more, however many prompts there are and whatever the type (their lengths
// may be equal).
static int check_general_splits()
{
    for (int dtype : {SPD_F32, SPD_BF16})
        for (int D : {64, 96})
            for (int groups : {1, 2, 3, 8, 16})
                for (long long len : {512ll, 2048ll, 8192ll}) {
                    spd_attn_desc d = {dtype, 32, 8, D, groups, 64, (64 + groups - 1) / groups, 0, 0.f, 0};
                    Plan pl;
                    if (make_plan(&d, len, 100, &pl) != SPD_OK)
                        return fail("make_plan refused a valid description", groups, len);
                    const int block = rows_per_block(D, 4ll * d.max_samples_per_prompt);
                    const long long units = 8ll * groups * ((4 * d.max_samples_per_prompt + block - 1) / block);
                    if ((pl.num_prefix_splits - 1) * units >= 256)
                        return fail("more workgroups than CUs", units, pl.num_prefix_splits);
                }
    return 0;
}

// Chunks shorter than eight tiles, or shared by wavefronts, do not go through LDS; nor do other types and widths.
static int check_rows_through_lds()
{
    for (int chunk : {64, 96, 192, 224, 256, 320, 768})
        for (int share : {1, 2, 4})
            for (int D : {56, 64, 96})
                for (int dtype : {SPD_F32, SPD_BF16})
                    if (rows_through_lds(dtype, D, chunk, share) != (dtype == SPD_BF16 && D == 64 && share == 1 && chunk >= 256))
                        return fail("rows through LDS", chunk, share);
    return 0;
}

// Just below and just above each line of a plain tiled call (8 KV heads, one prompt).
static int check_lines()
{
    struct Line {
        int samples, q_heads;
        long long prefix, suffix;
        int split_tokens, splits, chunk_tokens, chunks;
        bool folds;
    };
    const Line lines[] = {
        // the stream, by its bound, outlasts a pass of 128 workgroups (33 x suffix x 0.85 tokens, 1343 of them a us)
        {33, 16, 3000, 492, 128, 24, 64, 8, true}, {33, 16, 3000, 493, 192, 16, 64, 8, false},
        // whose splits hold 512 tokens
        {33, 16, 8192, 940, 512, 16, 96, 10, false}, {33, 16, 8193, 940, 320, 26, 96, 10, true},
        // the bound allows for a stream beside which two splits are taken together
        {64, 32, 8192, 489, 512, 16, 96, 6, false}, {64, 32, 8192, 490, 512, 16, 96, 6, true},
        // one split only
        {1024, 32, 4096, 700, 4096, 1, 704, 1, false},
        // 2048 and 2040 (sample, KV head) pairs
        {256, 16, 300, 700, 128, 3, 704, 1, false}, {255, 16, 300, 700, 128, 3, 320, 3, false},
    };
    for (const Line& x : lines) {
        spd_attn_desc d = {SPD_BF16, x.q_heads, 8, 128, 1, x.samples, x.samples, 0, 0.f, 0};
        Plan pl;
        if (make_plan(&d, x.prefix, x.suffix, &pl) != SPD_OK)
            return fail("make_plan refused a valid description", x.prefix, x.suffix);
        if (pl.prefix_split_tokens != x.split_tokens || pl.num_prefix_splits != x.splits)
            return fail("prefix splits at a line", pl.prefix_split_tokens, pl.num_prefix_splits);
        if (pl.suffix_chunk_tokens != x.chunk_tokens || pl.num_suffix_chunks != x.chunks)
            return fail("suffix chunks at a line", pl.suffix_chunk_tokens, pl.num_suffix_chunks);
        if ((pl.fold_tokens > 0.0) != x.folds)
            return fail("folded splits at a line", x.prefix, x.suffix);
    }
    spd_attn_desc d = {SPD_BF16, 1, 1, 128, 1, 2047, 2047, 0, 0.f, 0};
    if (plan_suffix_chunk(&d, 700) != 320 || (d.num_samples = 2048, plan_suffix_chunk(&d, 700)) != 704)
        return fail("chunks at 2048 pairs", 0, 0);
    return 0;
}

int main()
{
    if (check_lines())
        return 1;
    if (check_rows_through_lds())
        return 1;
    if (check_general_splits())
        return 1;
    if (check_stream())
        return 1;
    if (check_two_launches())
        return 1;
    if (check_suffix_order())
        return 1;
    const long long lens[] = {0, 1, 63, 64, 65, 97, 127, 129, 193, 257, 385, 769, 1025, 2048, 4097, 8192, 47104, 100000, 1ll << 30};
    const int samples[] = {1, 3, 16, 64, 191, 192, 255, 256, 1024, 1536, 2047, 100000};
    const int prompts[] = {1, 2, 8, 26};
    int checked = 0;
    for (int dtype : {SPD_F32, SPD_BF16})
        for (int D : {64, 128, 256})
            for (int g : {1, 4, 8, 16})
                for (int hkv : {1, 8})
                    for (int B : prompts)
                        for (int N : samples)
                            for (long long lp : lens)
                                for (long long ls : lens) {
                                    if (N < B)
                                        continue;
                                    spd_attn_desc d = {dtype, g * hkv, hkv, D, B, N, (N + B - 1) / B, 0, 0.f, 0};
                                    Plan pl;
                                    if (make_plan(&d, lp, ls, &pl) != SPD_OK)
                                        return fail("make_plan refused a valid description", lp, ls);
                                    if (lp > 0 && (pl.prefix_split_tokens <= 0 || pl.prefix_split_tokens % 64))
                                        return fail("split not a positive multiple of 64", lp, pl.prefix_split_tokens);
                                    if (ls > 0 && (pl.suffix_chunk_tokens < 64 || pl.suffix_chunk_tokens % 32))
                                        return fail("chunk not a multiple of 32", ls, pl.suffix_chunk_tokens);
                                    if (pl.num_prefix_splits > kMaxSplits || pl.num_suffix_chunks > kMaxSplits)
                                        return fail("more parts than the merge takes", pl.num_prefix_splits,
                                                    pl.num_suffix_chunks);
                                    if ((long long)pl.num_prefix_splits * pl.prefix_split_tokens < lp ||
                                        (long long)pl.num_suffix_chunks * pl.suffix_chunk_tokens < ls)
                                        return fail("parts do not cover the length", lp, ls);
                                    if (pl.num_prefix_splits > 0 &&
                                        (long long)(pl.num_prefix_splits - 1) * pl.prefix_split_tokens >= lp)
                                        return fail("an empty last split", lp, pl.prefix_split_tokens);
                                    // whatever the suffix bound: splits no longer than a workgroup per CU gives, or 512 tokens
                                    const int finest = plan_prefix_split(&d, B, (N + B - 1) / B, lp, kMaxSplits);
                                    if (pl.prefix_split_tokens > (finest > 512 ? finest : 512))
                                        return fail("splits grow with the suffix bound", finest, pl.prefix_split_tokens);
                                    if (pl.fold_tokens < 0.0 || (pl.fold_tokens > 0.0 && (pl.num_prefix_splits < 2 || !tiled(&d) ||
                                        pl.fold_tokens > (double)N * (double)ls)))
                                        return fail("splits folded in vain", lp, ls);
                                    const size_t slots = (size_t)pl.num_prefix_splits + pl.num_suffix_chunks;
                                    if (pl.acc_bytes < slots * N * d.num_q_heads * D * 4 || pl.acc_bytes % 256 ||
                                        pl.ml_bytes < slots * N * d.num_q_heads * 8 || pl.ml_bytes % 256)
                                        return fail("workspace too small or misaligned", (long long)pl.acc_bytes,
                                                    (long long)pl.ml_bytes);
                                    // what the size functions count covers the plan, part by part and in bytes
                                    const int splits = sized_prefix_splits(&d, lp), chunks = sized_suffix_chunks(&d, ls);
                                    if (splits < pl.num_prefix_splits || chunks < pl.num_suffix_chunks || chunks > kMaxSplits)
                                        return fail("more parts than the workspace is sized for", lp, ls);
                                    if (workspace_bytes(&d, 1, &lp, ls, state_bytes(&d, splits + chunks)) < pl.acc_bytes + pl.ml_bytes)
                                        return fail("reported size below the call's own need", lp, ls);
                                    // the same problem as a tree of one to four levels
                                    for (int levels = 1; levels <= SPD_MAX_PREFIX_LEVELS; ++levels) {
                                        spd_prefix_level lv[SPD_MAX_PREFIX_LEVELS] = {};
                                        for (int l = 0; l < levels; ++l) {
                                            lv[l].num_groups = l == 0 ? 1 : B;
                                            lv[l].max_samples_per_group = l == 0 ? 0 : (N + B - 1) / B;
                                            lv[l].max_len = l % 2 ? lp / 2 : lp;
                                        }
                                        LevelPlan lpn;
                                        if (make_level_plan(&d, levels, lv, ls, &lpn) != SPD_OK)
                                            return fail("make_level_plan refused a valid tree", levels, lp);
                                        int slots_seen = 0;
                                        for (int l = 0; l < levels; ++l) {
                                            if (lpn.slot0[l] != slots_seen)
                                                return fail("slot ranges not consecutive", l, lpn.slot0[l]);
                                            slots_seen += lpn.num_splits[l];
                                        }
                                        if (chunks < lpn.num_suffix_chunks ||
                                            state_bytes(&d, slots_seen + chunks) < lpn.acc_bytes + lpn.ml_bytes)
                                            return fail("a tree's need above its reported size", levels, ls);
                                        if (slots_seen > kMaxSplits || slots_seen + lpn.num_suffix_chunks != lpn.num_slots)
                                            return fail("slot count", slots_seen, lpn.num_slots);
                                    }
                                    ++checked;
                                }
    // refusals
    spd_attn_desc bad = {SPD_BF16, 7, 2, 128, 1, 4, 0, 0, 0.f, 0};
    Plan pl;
    if (make_plan(&bad, 10, 10, &pl) != SPD_EINVAL || make_plan(nullptr, 1, 1, &pl) != SPD_EINVAL)
        return fail("invalid description accepted", 0, 0);
    spd_attn_desc ok = {SPD_BF16, 8, 2, 128, 1, 4, 0, 0, 0.f, 0};
    if (make_plan(&ok, -1, 0, &pl) != SPD_EINVAL || make_plan(&ok, (1ll << 30) + 1, 0, &pl) != SPD_EINVAL)
        return fail("invalid bound accepted", 0, 0);
    LevelPlan lpn;
    if (make_level_plan(&ok, 0, nullptr, 0, &lpn) != SPD_EINVAL)
        return fail("empty tree accepted", 0, 0);
    std::printf("ok: %d plans\n", checked);
    return 0;
}
