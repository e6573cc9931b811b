// Launch planning of the attention calls: host arithmetic only (no HIP, no allocation), so that it
// can also be compiled and exercised on a machine without a GPU.
//
// A call is cut into prefix splits (one workgroup per (group, KV head, row tile, split)) and suffix
// chunks (one wavefront per (sample, KV head, chunk)); every (split | chunk) owns one slot of
// partial softmax state per output row, which the merge combines.
#pragma once

#include "../../include/spdecode.h"

#include <stddef.h>
#include <stdint.h>

namespace spd {
namespace plan {

struct Plan {
    int prefix_split_tokens, num_prefix_splits;
    int suffix_chunk_tokens, num_suffix_chunks;
    double fold_tokens;  // suffix tokens from which a prefix workgroup takes two splits (0: never)
    size_t acc_bytes, ml_bytes;
};

// Plan of a multi-level call: split size and count per level, slot offsets, suffix chunks.
struct LevelPlan {
    int split_tokens[SPD_MAX_PREFIX_LEVELS], num_splits[SPD_MAX_PREFIX_LEVELS], slot0[SPD_MAX_PREFIX_LEVELS];
    int suffix_chunk_tokens, num_suffix_chunks, num_slots;
    double fold_tokens;
    size_t acc_bytes, ml_bytes;
};

constexpr int kPrefixBlockRows = 128;  // query rows per prefix workgroup on the tiled path
constexpr int kMaxSplits = 64;         // the merge takes 64 prefix splits and 64 suffix chunks
constexpr long long kMaxLen = 1ll << 30;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline int check_desc(const spd_attn_desc* d)
{
    if (!d)
        return SPD_EINVAL;
    if (d->num_q_heads <= 0 || d->num_kv_heads <= 0 || d->head_dim <= 0 || d->num_prompts <= 0 ||
        d->num_samples <= 0 || d->max_samples_per_prompt < 0)
        return SPD_EINVAL;
    if (d->num_q_heads % d->num_kv_heads != 0)
        return SPD_EINVAL;
    if (d->dtype != SPD_F32 && d->dtype != SPD_BF16)
        return SPD_EUNSUPPORTED;
    if (d->page_size != 0 && d->page_size != 16)
        return SPD_EUNSUPPORTED;
    if (d->head_dim > 256 || d->head_dim % 8 != 0)
        return SPD_EUNSUPPORTED;
    if (d->stages & ~(uint32_t)(SPD_STAGE_PREFIX | SPD_STAGE_SUFFIX | SPD_STAGE_MERGE))
        return SPD_EINVAL;
    return SPD_OK;
}

// Tokens per part so that at most `max_parts` parts cover `len`, in multiples of `quantum`.
inline int part_tokens(long long len, int min_tokens, int max_parts, int quantum)
{
    long long t = (len + max_parts - 1) / max_parts;
    if (t < min_tokens)
        t = min_tokens;
    t = (t + quantum - 1) / quantum * quantum;
    return (int)t;
}

// Query rows per wavefront of the general kernel (fp32, other head dimensions): 32 use every loaded K and
// V register twice; 16 when there are no more rows than that, or when two blocks' queries and
// accumulators would not leave room for two wavefronts per SIMD (more than 64 channels).
inline int rows_per_block(int head_dim, long long rows) { return rows > 16 && head_dim <= 64 ? 32 : 16; }

// Fewest tokens per split in the general kernel: a tile or more for each of four wavefronts.
inline int min_split_tokens(const spd_attn_desc* d) { return d->dtype == SPD_BF16 ? 128 : 64; }

inline bool tiled(const spd_attn_desc* d) { return d->dtype == SPD_BF16 && d->head_dim == 128; }

// Workgroups of 128 rows, independent of the splits, that a prefix level of the tiled path has.
inline long long prefix_units(const spd_attn_desc* d, int groups, int spp)
{
    const long long rows = (long long)spp * (d->num_q_heads / d->num_kv_heads);
    return (long long)groups * d->num_kv_heads * ((rows + kPrefixBlockRows - 1) / kPrefixBlockRows);
}

// The prefix and suffix passes of a tiled call share a launch up to 16 query heads per KV head (the columns of the suffix
// pass's product) and 65535 (group, KV head) pairs.
inline bool one_launch(const spd_attn_desc* d, int groups)
{
    return tiled(d) && d->num_q_heads <= 16 * d->num_kv_heads && (long long)groups * d->num_kv_heads <= 65535;
}

// us that a prefix workgroup beside the suffix stream takes for `tokens` tokens: 0.9 a 32-token tile, 5 before the first.
inline double prefix_time(long long tokens) { return 5.0 + 0.9 * (double)tokens / 32.0; }

// Suffix tokens that the stream takes `us` for (5.5 TB/s, bf16, 128 channels).
inline double stream_tokens(const spd_attn_desc* d, double us) { return us * 5.5e6 / (512.0 * d->num_kv_heads); }

// Workgroups that the prefix pass of a plain call should have on the tiled path: one per CU, or half as many where their
// splits hold no more than 512 tokens and the suffix stream, by the call's bounds, lasts longer: every workgroup
// less is a place for four wavefronts that stream, and a partial state less per row.  The bound says little about the
// lengths (a slot's capacity, of which a step may use a tenth), so the line lies where the pass alone takes as long
// either way.  256 / 128 / 64 workgroups, at 20 to 60, 100 to 300 and 500 to 1000 tokens of a bound of 1024: 32 samples of
// an 8k prompt (512 tokens in 128) 22.6 / 22.9 / 30.3, 24.3 / 25.6 / 32.5, 38.4 / 35.1 / 38.8 us, 64 samples of a 3k
// prompt (384) 20.0 / 20.4 / 25.7, 28.3 / 24.4 / 29.3, 49.9 / 44.6 / 47.7, 256 samples of a 1k prompt (512)
// 27.1 / 25.3 / 33.8, 60.7 / 56.2 / 50.5, 155 / 145 / 138; but 64 samples of an 8k prompt (1024) 26.5 / 32.6 / 48.8,
// 29.9 / 35.6 / 51.8, 51.3 / 51.6 / 61.1: see fold_tokens.
constexpr int kHalfSplitTokens = 512;

inline int prefix_workgroups(const spd_attn_desc* d, int groups, int spp, long long max_prefix, long long max_suffix)
{
    if (!one_launch(d, groups) || max_prefix == 0)
        return 256;
    const long long base = prefix_units(d, groups, spp), splits = (128 + base - 1) / base;
    const long long tokens = (max_prefix + splits - 1) / splits;
    const bool longer = (double)d->num_samples * (double)max_suffix * 0.85 >= stream_tokens(d, prefix_time(tokens));
    return tokens <= kHalfSplitTokens && longer ? 128 : 256;
}

// Longer splits are put together on the device, where the lengths are: a workgroup of the fused launch takes two splits,
// and the other one of the two ends at once, where the suffixes hold this many tokens (two splits take no
// more than 1.45 of the stream's time).  0: never.  One split / two / as the tokens say, 64 samples of an 8k prompt,
// suffixes up to 50, 300, 600, 1000 tokens, bound 2048: 27.1 / 32.0 / 27.3, 35.3 / 33.1 / 35.2, 38.6 / 39.9 / 38.9,
// 55.0 / 45.5 / 47.0 us; 96 samples, 128 to 1024 tokens 72.2 / 63.4 / 61.7; 128 samples of a 4k prompt at 300 to 600 of 1024
// lose 54.1 / 55.9 / 58.4, at 500 to 1000 of 2048 stay 86.3 / 83.2 / 86.3.  To read the lengths costs a call 0.3 us.
inline double fold_tokens(const spd_attn_desc* d, int groups, int split_tokens, int splits, int workgroups, long long max_suffix)
{
    if (!one_launch(d, groups) || splits < 2 || workgroups < 256)
        return 0.0;
    const double tokens = stream_tokens(d, prefix_time(2ll * split_tokens) / 1.45);
    return (double)d->num_samples * (double)max_suffix >= tokens ? tokens : 0.0;
}

// Tokens per split of a prefix level with `groups` groups of at most `spp` samples and lengths up to
// `max_prefix`, at most `max_splits` splits.
inline int plan_prefix_split(const spd_attn_desc* d, int groups, int spp, long long max_prefix, int max_splits,
                             int workgroups = 256)
{
    if (tiled(d)) {
        // one workgroup per (group, KV head, row tile, split), in multiples of the 64-token tile
        const long long base = prefix_units(d, groups, spp);
        long long want = (workgroups + base - 1) / base;
        if (want > max_splits) want = max_splits;
        long long t = (max_prefix + want - 1) / want;
        t = (t + 63) / 64 * 64;
        if (t < 128) t = 128;  // at least two tiles per split: a one-tile workgroup is all start-up
        return (int)t;
    }
    // general kernel: enough splits for a workgroup per CU, a tile or more per wavefront.  (bf16, 64 channels, 1.5 per CU
    // for several prompts: where their lengths differ 2 prompts of 500 to 4000 tokens x 128 samples 42.0 -> 36 us, 3 x 21
    // 25.0 -> 22.3, but of equal lengths 16 prompts of 512 x 4 10.6 -> 14.0, 8 of 1024 x 8 13.3 -> 15.3, 2 of 2048
    // x 128 50.0 -> 58.4: the lengths are on the device.)
    const long long rows = (long long)spp * (d->num_q_heads / d->num_kv_heads);
    const int block = rows_per_block(d->head_dim, rows);
    const long long base = (long long)groups * d->num_kv_heads * ((rows + block - 1) / block);
    const long long want = (256 + base - 1) / base;
    return part_tokens(max_prefix, min_split_tokens(d), (int)(want > max_splits ? max_splits : want), 64);
}

// From how many bytes of KV (by the call's bounds) the suffix pass marks V as streamed: three quarters of the last-level
// cache's 256 MB.  Where such buffers (layers, or batches) are taken in turn, leaving V out of the cache saves the cache's own
// traffic; a single buffer that every step reads again loses what it kept there.  Not marked / marked, us, three
// buffers in turn | the same one, bounds in MB, tokens present in parentheses: 138 MB (half) 25.9 / 26.0 | 24.7 / 25.9, paged
// 25.8 / 26.7 | 25.2 / 26.9; 172 MB (half) 30.1 / 29.0 | 26.4 / 28.5; 205 MB (half) 34.5 / 30.8 | 29.7 / 30.5, (three
// quarters) 44.1 / 39.4 | 36.3 / 37.1; 272 MB (half) 46.9 / 42.2 | 38.0 / 40.1; 340 MB (nine tenths) 73.4 / 68.6 | 60.5 / 57.2; 1 GB
// (a tenth) 36.6 / 33.6 | 31.5 / 32.4.  Below the line what a repeated buffer loses made such calls slower than they were
// with neither whole-line K loads nor streaming (25.1 and 27.8 us at 138 and 172 MB).
constexpr double kStreamBytes = 192.0 * 1024 * 1024;
// K too from 1 GiB on, and only of contiguous KV.  V only / both, in turn | the same one: 416 samples, a tree (1.7 GiB by its
// bounds, 1 GB present) 241.7 / 235.0 | 240.7 / 226.7, 2000 samples (2.5 GB, two thirds) 318.8 / 302.2 | 323.8 / 305.5, 256 samples
// (1.1 GB, half) 125.9 / 119.3 | 118.4 / 118.7, 128 samples at 100 to 200, 200 to 400, 400 to 800 of 4096 tokens
// 34.4 / 32.3 | 32.4 / 32.3, 44.4 / 42.1 | 40.1 / 42.1, 72.1 / 68.5 | 62.7 / 67.0 (the last two before
// any streaming, in other chunks: 64.6, 92.1 | 54.6, 77.9).  At 0.9 GiB in turn -3 to -5 %, the same one +2 to +4 %.  To let the
// lengths decide costs every wavefront a round trip (2000 samples at up to 30 tokens 76 -> 87).
constexpr double kStreamKBytes = 1024.0 * 1024 * 1024;

inline int plan_stream(const spd_attn_desc* d, int num_levels, const spd_prefix_level* levels, long long max_suffix)
{
    double tokens = (double)d->num_samples * (double)max_suffix;
    for (int l = 0; l < num_levels; ++l)
        tokens += (double)levels[l].num_groups * (double)levels[l].max_len;
    const double bytes = 2.0 * tokens * d->num_kv_heads * d->head_dim * (d->dtype == SPD_BF16 ? 2 : 4);
    if (bytes < kStreamBytes)
        return 0;
    return bytes >= kStreamKBytes && d->page_size == 0 ? 2 : 1;
}

// Sample and chunk of suffix unit `unit` (a suffix item without its KV head, which runs fastest).  Units go chunk
// after chunk through all samples, so that with ragged lengths the chunks that are mostly empty come last, and
// an even number of samples starts every chunk one sample further on.  Workgroups go to the eight XCDs in turn: where
// the samples' workgroups of a chunk are a multiple of eight, all chunks of a sample would else be on the same ones
// (24 samples x 8 KV heads, 512 to 1024 tokens, prompt of 1k: 25.5 us, turned 22.4); turned, a sample's next chunk is
// an odd number of samples on.  In sample-major order, where a sample has 8 or 16 workgroups, all last chunks
// are on the same ones (128 samples x 8 heads, up to 1024 tokens beside a prompt of 4k: 96 us, 70).
struct SuffixPlace {
    int n, chunk;
};
constexpr SuffixPlace suffix_place(unsigned unit, unsigned samples)
{
    const unsigned chunk = unit / samples;
    const unsigned place = unit - chunk * samples;
    return {(int)(samples % 2 ? place : (place + chunk) % samples), (int)chunk};
}

// From how many (sample, KV head) pairs the chunks alone fill the chip's 2048 wavefront places.
constexpr long long kManyPairs = 2048;

inline bool many_suffixes(const spd_attn_desc* d) { return (long long)d->num_samples * d->num_kv_heads >= kManyPairs; }

// Tokens per chunk for about a place per (pair, chunk) item: 64 to 320.  (96 and 192 in place of 128 and 256: in the items'
// order neither is the better one throughout.  192 / 256, us, up to 1024 tokens of 8 KV heads: 64 samples of an 8k
// prompt at 150 to 300 30.3 / 32.5, 300 to 600 47.9 / 37.5, 500 to 1000 50.7 / 51.5, 32 samples 24.7 / 31.7, 37.3 / 32.7.)
inline long long short_chunk(const spd_attn_desc* d, long long max_suffix)
{
    const long long pairs = (long long)d->num_samples * d->num_kv_heads;
    const long long want_chunks = (2048 + pairs - 1) / pairs;
    long long t = (max_suffix + want_chunks - 1) / want_chunks;
    t = (t + 63) / 64 * 64;
    if (t < 64) t = 64;
    if (t > 320) t = 320;
    return t == 128 || t == 256 ? t / 4 * 3 : t;
}

// Tokens per suffix chunk, at most kMaxSplits chunks.
//   Fewer pairs than places: enough (pair, chunk) items to fill them, chunks of 64 to 320 tokens.
//   More: as few equal parts as chunks of up to 768 tokens allow: a chunk pays some 4 us
//   before its first tile is there and leaves a partial state.  8 prompts x 128 samples, up to 2048 tokens, 320 tokens
//   861 us, 416 840, 512 825, 640 817, 768 801, 1024 807; 416 samples x 8 heads, up to 1024 tokens, beside a
//   tree of prefixes: 320 264, 512 257, 640 257, 768 266, 1024 279.
inline int plan_suffix_chunk(const spd_attn_desc* d, long long max_suffix)
{
    long long t;
    if (many_suffixes(d)) {
        const long long parts = max_suffix > 768 ? (max_suffix + 767) / 768 : 1;
        t = ((max_suffix + parts - 1) / parts + 31) / 32 * 32;
        if (t < 64) t = 64;
    } else {
        t = short_chunk(d, max_suffix);
    }
    if (max_suffix > t * kMaxSplits) t = part_tokens(max_suffix, 64, kMaxSplits, 64);
    return (int)t;
}

// Whether the general kernel takes bf16 with 64 channels through LDS, two tiles ahead: where a wavefront has a suffix
// chunk of eight tiles or more to itself.  Fewer tiles do not pay back the way through LDS, and its 64 KB leave two
// workgroups on a CU (registers: four where a wavefront has 16 query rows, two where it has 32).  Registers / LDS, us: 4 prompts x 100 samples at up to 256, 501, 1000
// tokens 48.8 / 47.4, 67.5 / 62.3, 117.6 / 112.3, 2 x 128 at 256 to 512 64.2 / 59.2, 1 x 300 at up to 1000 83.9 / 80.4; 16 prompts x 4
// samples at up to 256 (64-token chunks) 15.2 / 18.0, 4 x 16 at 256 to 512 (96) 27.0 / 29.1, 8 x 8 22.6 / 24.4, 3 x 21
// at up to 501 25.3 / 26.2, 64 x 1 at up to 1000 (192) 29.9 / 31.0, 32 x 8 at up to 64 18.9 / 20.1.
inline bool rows_through_lds(int dtype, int head_dim, int chunk_tokens, int share)
{
    return dtype == SPD_BF16 && head_dim == 64 && share == 1 && chunk_tokens >= 256;
}

// ---- workspace sizes -----------------------------------------------------------------------------------
// A program allocates once, for its largest batch and its longest lengths.  Split counts fall in steps as
// rows are added, so a call's own need is not monotone; what the size functions report is the most
// that any call of no more samples, however grouped, and no longer lengths can need.  (On the bf16 /
// head_dim 128 path they report what this one call needs in the finest plan: splits of a workgroup per CU and short
// chunks.)  Suffixes are counted in the chunks of short_chunk, of
// which plan_suffix_chunk never makes more: the longer chunks of many pairs are no help to smaller batches.
inline int sized_suffix_chunks(const spd_attn_desc* d, long long max_suffix)
{
    long long t = short_chunk(d, max_suffix);
    if (max_suffix > t * kMaxSplits) t = part_tokens(max_suffix, 64, kMaxSplits, 64);
    return (int)((max_suffix + t - 1) / t);
}

// Prefix splits that a workspace is sized for: those of a workgroup per CU.
inline int sized_prefix_splits(const spd_attn_desc* d, long long max_prefix)
{
    const int spp = d->max_samples_per_prompt > 0 ? d->max_samples_per_prompt : d->num_samples;
    const int t = plan_prefix_split(d, d->num_prompts, spp, max_prefix, kMaxSplits);
    return (int)((max_prefix + t - 1) / t);
}

// Most suffix chunks that `samples` samples with suffixes of up to `max_suffix` tokens are cut into: the count
// is largest at `max_suffix`, where a chunk size stops being used, or where it reaches kMaxSplits chunks.
inline int most_suffix_chunks(const spd_attn_desc* d, long long samples, long long max_suffix)
{
    spd_attn_desc t = *d;
    t.num_samples = (int)samples;
    const long long pairs = samples * d->num_kv_heads, want = (2048 + pairs - 1) / pairs;
    long long most = 0;
    auto at = [&](long long len) {
        len = len < max_suffix ? len : max_suffix;
        const long long n = sized_suffix_chunks(&t, len);
        most = n > most ? n : most;
    };
    at(max_suffix);
    for (int k = 1; k <= 5; ++k) {
        at(64 * k * want);
        at(64ll * k * kMaxSplits);
    }
    at(96ll * kMaxSplits);
    return (int)most;
}

// Most splits of a prefix level of up to `max_len` tokens that `samples` samples share.  One group takes the
// fewest row blocks, so it is cut into the most splits.
inline int most_prefix_splits(const spd_attn_desc* d, long long samples, long long max_len, int max_splits)
{
    const long long rows = samples * (d->num_q_heads / d->num_kv_heads);
    const int block = rows_per_block(d->head_dim, kPrefixBlockRows);  // the larger of the two blocks
    const long long base = (long long)d->num_kv_heads * ((rows + block - 1) / block);
    long long want = (256 + base - 1) / base;
    want = want > max_splits ? max_splits : want;
    const int least = min_split_tokens(d);
    const long long splits = (max_len + least - 1) / least;
    return (int)(splits < want ? splits : want);
}

// Bytes of `slots` partial states for every output row.
inline size_t state_bytes(const spd_attn_desc* d, long long slots)
{
    const size_t rows = (size_t)d->num_samples * d->num_q_heads * (size_t)slots;
    return align_up(rows * d->head_dim * sizeof(float), 256) + align_up(rows * 2 * sizeof(float), 256);
}

// Bytes to report for a call of d->num_samples samples with prefix levels of up to max_len[] tokens; `own` is
// what the call itself needs (with sized_suffix_chunks).
inline size_t workspace_bytes(const spd_attn_desc* d, int num_levels, const long long* max_len, long long max_suffix,
                              size_t own)
{
    if (d->dtype == SPD_BF16 && d->head_dim == 128)
        return own;
    auto slots = [&](long long samples) {
        long long n = most_suffix_chunks(d, samples, max_suffix);
        for (int l = 0; l < num_levels; ++l)
            n += most_prefix_splits(d, samples, max_len[l], kMaxSplits / num_levels);
        return n;
    };
    // the largest samples * slots(samples) of all batches up to this one; slots() only falls, so the
    // batches that count are the last ones before it falls
    const long long top = slots(1);
    long long most = 0;
    for (long long n = d->num_samples; n > 0 && n * top > most;) {
        const long long s = slots(n);
        most = n * s > most ? n * s : most;
        long long more = 0, same = n;  // slots(more) > s (or more == 0), slots(same) == s
        while (same - more > 1) {
            const long long mid = (more + same) / 2;
            (slots(mid) > s ? more : same) = mid;
        }
        n = more;
    }
    const size_t acc = align_up((size_t)most * d->num_q_heads * d->head_dim * sizeof(float), 256);
    const size_t ml = align_up((size_t)most * d->num_q_heads * 2 * sizeof(float), 256);
    return acc + ml > own ? acc + ml : own;
}

inline int make_plan(const spd_attn_desc* d, long long max_prefix, long long max_suffix, Plan* pl)
{
    const int rc = check_desc(d);
    if (rc != SPD_OK)
        return rc;
    if (max_prefix < 0 || max_suffix < 0 || max_prefix > kMaxLen || max_suffix > kMaxLen)
        return SPD_EINVAL;
    const int spp = d->max_samples_per_prompt > 0 ? d->max_samples_per_prompt : d->num_samples;
    const int workgroups = prefix_workgroups(d, d->num_prompts, spp, max_prefix, max_suffix);
    pl->prefix_split_tokens = plan_prefix_split(d, d->num_prompts, spp, max_prefix, kMaxSplits, workgroups);
    pl->num_prefix_splits = (int)((max_prefix + pl->prefix_split_tokens - 1) / pl->prefix_split_tokens);
    pl->fold_tokens = fold_tokens(d, d->num_prompts, pl->prefix_split_tokens, pl->num_prefix_splits, workgroups, max_suffix);
    pl->suffix_chunk_tokens = plan_suffix_chunk(d, max_suffix);
    pl->num_suffix_chunks = (int)((max_suffix + pl->suffix_chunk_tokens - 1) / pl->suffix_chunk_tokens);
    const size_t rows = (size_t)d->num_samples * d->num_q_heads;
    const size_t slots = (size_t)pl->num_prefix_splits + pl->num_suffix_chunks;
    pl->acc_bytes = align_up(slots * rows * d->head_dim * sizeof(float), 256);
    pl->ml_bytes = align_up(slots * rows * 2 * sizeof(float), 256);
    return SPD_OK;
}

inline int make_level_plan(const spd_attn_desc* d, int num_levels, const spd_prefix_level* levels, long long max_suffix,
                           LevelPlan* lp)
{
    if (!d || num_levels < 1 || num_levels > SPD_MAX_PREFIX_LEVELS || !levels)
        return SPD_EINVAL;
    Plan pl;
    spd_attn_desc tmp = *d;
    tmp.num_prompts = 1;
    tmp.max_samples_per_prompt = 0;
    const int rc = make_plan(&tmp, 0, max_suffix, &pl);  // validates desc and plans the suffix chunks
    if (rc != SPD_OK)
        return rc;
    lp->suffix_chunk_tokens = pl.suffix_chunk_tokens;
    lp->num_suffix_chunks = pl.num_suffix_chunks;
    lp->fold_tokens = 0.0;
    const int max_splits = kMaxSplits / num_levels;  // the merge takes kMaxSplits prefix splits in all
    int slots = 0;
    for (int l = 0; l < num_levels; ++l) {
        const spd_prefix_level& L = levels[l];
        if (L.num_groups < 1 || L.max_samples_per_group < 0 || L.max_len < 0 || L.max_len > kMaxLen)
            return SPD_EINVAL;
        const int spp = L.max_samples_per_group > 0 ? L.max_samples_per_group : d->num_samples;
        lp->split_tokens[l] = plan_prefix_split(d, L.num_groups, spp, L.max_len, max_splits);
        lp->num_splits[l] = (int)((L.max_len + lp->split_tokens[l] - 1) / lp->split_tokens[l]);
        lp->slot0[l] = slots;
        slots += lp->num_splits[l];
    }
    lp->num_slots = slots + lp->num_suffix_chunks;
    const size_t rows = (size_t)d->num_samples * d->num_q_heads;
    lp->acc_bytes = align_up((size_t)lp->num_slots * rows * d->head_dim * sizeof(float), 256);
    lp->ml_bytes = align_up((size_t)lp->num_slots * rows * 2 * sizeof(float), 256);
    return SPD_OK;
}

}  // namespace plan
}  // namespace spd
