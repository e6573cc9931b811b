// Prefix (cascade) pass (bf16, head_dim 128): all samples' queries of one KV head form
// a dense row tile against the shared prompt KV, so the prompt is read once per row
// tile instead of once per sample.
//
// Workgroup = (prompt b, KV head j, tile of 32*WAVES query rows, split of the prefix); WAVES is 4
// or 8.
// A query row is (sample, head in group); each wavefront owns 32 rows (one 32-wide column
// block of the transposed products).
//
// Data movement.  K and V tiles of 32 tokens go from global memory straight into LDS
// (global_load_lds_dwordx4, no registers in between), into a ring of five K slots and a ring of five V
// slots, four tiles ahead of their use.  Both tiles are row-major [token][256 bytes] without
// padding; bank conflicts are avoided by an XOR swizzle of the 16-byte pieces of a row,
// applied on the global side of the copy (lane L of a copy instruction always lands at
// LDS offset 16 L, but it may fetch any piece).
//   K  read with ds_read_b128 as the A operand of S^T = K Q^T
//      (v_mfma_f32_32x32x16_bf16, B = query rows held in registers);
//   V  read with the transposing ds_read_b64_tr_b16 (each lane receives four tokens of one
//      channel) as the A operand of O^T += V^T P^T, B = P, which is the S^T accumulator
//      itself repacked to bf16.
// The LDS reads are issued by hand (inline assembly) a few fragments ahead of the MFMA that
// consumes them, with exact lgkmcnt waits; the compiler's own wait insertion would otherwise
// drain every outstanding copy before any LDS read.
//
// Every lane owns one query row in both products, so the online-softmax statistics and the
// accumulator rescale are lane-local.  The running state is the deferred-division form of the
// paper's online-softmax recurrence (App., attn task 2).
//
// Bound: the matrix pipe (16 products a tile and wavefront at about 25 ns each under load, i.e. near the
// 1.2 PFLOP/s that a large matrix product reaches on this card) and about 9 us of launch, first copies and the
// partial states.  Three tiles are in work at once, the scores of one, the softmax of the one before
// and P V of the one before that, interleaved instruction by instruction, because a wavefront is alone
// on its SIMD here (or beside a streaming one).  Measured against 64-token tiles with copies one tile
// ahead and the softmax between two MFMA regions, launches back to back: own launch, 8 prompts x 128 samples
// (longest split 13k tokens) 331 -> 260 us, 32 samples x 8 heads of a 16k prompt 34.5 -> 29.1; with the suffix
// pass in the launch, the latter 44.6 -> 41.4, 64 samples of an 8k prompt 54.5 -> 53.0.  Tried without
// gain: the two halves of a workgroup in opposite phases (products / softmax, own launch of the second
// shape 5 % slower), 64 KB of copies under way instead of 32 alone, five or seven LDS fragments ahead
// instead of four, tile orders rotated from split to split.
#pragma once

#include "spd_internal.h"

#include <hip/hip_fp16.h>

#include <utility>

namespace spd {
namespace prefix_impl {


typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kD = 128;
constexpr int kTileN = 32;               // tokens per tile
constexpr int kTileBytes = kTileN * 256;  // one K or V tile
constexpr int kRowU4 = kD * 2 / 16;
constexpr int kAhead = 4;                // LDS fragments in flight ahead of the MFMAs

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return *reinterpret_cast<bf16x8*>(&v); }
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return *reinterpret_cast<bf16x8*>(&v); }

// Two floats to packed bf16 (round to nearest even): one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16_rne(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    const bf16x2 r = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<const uint32_t*>(&r);
}

// Swizzle of the 16-byte pieces of token row `tok` (within a tile): piece p lives in slot
// p ^ swz(tok).  Sixteen consecutive rows get sixteen different values (K operand reads: 16
// lanes, 16 rows, one piece each), and four consecutive rows land in four different 64-byte
// quarters of the 256-byte bank window (V reads: four rows, up to four neighbouring pieces each).
__device__ __forceinline__ int swz(int tok) { return ((tok & 3) << 2) | ((tok >> 2) & 3); }

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    // vmcnt(N); expcnt and lgkmcnt left alone
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// One LDS fragment: a K fragment is one ds_read_b128, a V fragment two transposing reads.
// QK: a = channel step (0..7).  PV: a = token step (0..1), b = channel block (0..3).  When a region
// holds both products they alternate.
template <bool QK, bool PV, int K> struct Frag {
    static constexpr bool both = QK && PV;
    static constexpr int idx = both ? (K >> 1) : K;
    static constexpr bool is_pv = both ? ((K & 1) != 0) : PV;
    static constexpr int a = is_pv ? (idx >> 2) : idx;
    static constexpr int b = is_pv ? (idx & 3) : 0;
};
template <bool QK, bool PV> constexpr int frag_count() { return (QK ? 8 : 0) + (PV ? 8 : 0); }
// LDS instructions issued after fragment K while K is the oldest outstanding one
template <bool QK, bool PV, int K> constexpr int ops_after()
{
    int n = 0;
    for (int j = K + 1; j <= K + kAhead && j < frag_count<QK, PV>(); ++j) {
        const bool both = QK && PV;
        const bool is_pv = both ? ((j & 1) != 0) : PV;
        n += is_pv ? 2 : 1;
    }
    return n;
}

template <typename F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// The prefix level that the prefix fields of `p` describe.
__host__ __device__ inline PrefixLevelParams level_of(const AttnParams& p, int rowtiles)
{
    PrefixLevelParams lv;
    lv.k = p.k_prefix;
    lv.v = p.v_prefix;
    lv.lens = p.prefix_lens;
    lv.indptr = p.prefix_indptr;
    lv.pages = p.prefix_pages;
    lv.sample_indptr = p.sample_indptr;
    lv.split_tokens = p.prefix_split_tokens;
    lv.num_splits = p.num_prefix_splits;
    lv.slot0 = p.prefix_slot0;
    lv.rowtiles = rowtiles;
    lv.groups = p.B;
    return lv;
}

// Which (split, row tile, z = group * Hkv + KV head) the prefix workgroup with index `local` of a
// level takes.  Workgroups go to the eight XCDs in turn (index mod 8), and every XCD has an L2 of
// its own: the row tiles of one (split, z) read the same K and V, so they are given indices that
// agree mod 8 and follow one another, which puts them on one XCD at the same time (the prompt is
// then fetched into one L2 once instead of into as many L2s as there are row tiles).  That
// takes a number of (split, z) units divisible by 8; otherwise the split runs fastest, then the
// row tile, then z.
struct PrefixItem {
    int split, rowtile, z;
};
// The split that a unit of index u (u % num_splits counted around) takes: where num_splits shares a factor with
// the eight XCDs, u % num_splits alone would give an XCD the same splits of every prompt, and those past the
// end of the shorter prompts are empty (fp32, 3 prompts of 3003 .. 10880 tokens x 79 samples, four splits: 345 us
// against 269 with two).
__device__ __forceinline__ int turned_split(int u, int num_splits)
{
    if (num_splits & 1)
        return u % num_splits;
    // (constant over the splits of a unit's prompt in either case, so that every split is taken once)
    const int turn = num_splits == 2 || num_splits == 4 ? u >> 3 : u / num_splits;
    return (int)((unsigned)(u + turn) % (unsigned)num_splits);
}

__device__ __forceinline__ PrefixItem prefix_item(int local, int num_splits, int rowtiles, int zs)
{
    PrefixItem it;
    const int units = num_splits * zs;
    if (rowtiles > 1 && (units & 7) == 0) {
        const int slot = local >> 3;
        const int u = (local & 7) + 8 * (slot / rowtiles);
        it.rowtile = slot % rowtiles;
        it.split = turned_split(u, num_splits);
        it.z = u / num_splits;
    } else {
        it.split = turned_split(local, num_splits);
        const int rest = local / num_splits;
        it.rowtile = rest % rowtiles;
        it.z = rest / rowtiles;
    }
    return it;
}

// Copies of a tile start kCopyAhead tiles before its use; a ring holds the tile in use and those under way.
constexpr int kCopyAhead = 4;
constexpr int kRing = kCopyAhead + 1;
// LDS of a workgroup: the K ring followed by the V ring.
constexpr int kPrefixLds = 2 * kRing * kTileBytes;

// Body of one workgroup of WAVES wavefronts for prefix level `lv`: (split, rowtile,
// z = group * Hkv + KV head); `folded`: the even ones of two splits take both, the odd ones are empty.  `lds` is
// kPrefixLds bytes of LDS; every wavefront of the workgroup must call it (it uses workgroup barriers).
template <int WAVES, bool PAGED>
__device__ __forceinline__ void prefix_body(const AttnParams& p, const PrefixLevelParams& lv, uint4* lds, int split,
                                            int rowtile, int z, bool folded = false)
{
    constexpr int kIPW = 16 / WAVES;  // copy instructions per wave per step

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, h = lane >> 5;

    const int b = z / p.Hkv, j = z % p.Hkv;
    const int s0 = lv.sample_indptr[b];
    const int rows_b = (lv.sample_indptr[b + 1] - s0) * p.G;
    const int row0 = rowtile * 32 * WAVES;
    const int Lp = lv.lens[b];
    const int t0 = split * lv.split_tokens;
    const int t1 = min(Lp, t0 + (folded ? (split & 1 ? 0 : 2) : 1) * lv.split_tokens);
    if (row0 >= rows_b)
        return;
    if (t0 >= t1) {
        // empty split: l = 0 tells the merge to leave the slot out (its output part stays unwritten)
        const int rr = row0 + wave * 32 + col;
        if (rr < rows_b && h == 0)
            p.part_ml[part_index(p, (long long)(s0 + rr / p.G) * p.Hq + j * p.G + rr % p.G, lv.slot0 + split)] =
                make_float2(-INFINITY, 0.f);
        return;
    }

    const char* __restrict__ kg = (const char*)lv.k;
    const char* __restrict__ vg = (const char*)lv.v;
    // the page table is read with scalar loads (uniform index, constant address space)
    typedef const __attribute__((address_space(4))) int* const_int_ptr;
    const const_int_ptr pages = PAGED ? (const_int_ptr)(lv.pages + lv.indptr[b]) : nullptr;
    // byte strides of a token row and byte offset of token 0 of this KV head
    const long long tok_stride = PAGED ? 256 : (long long)p.Hkv * 256;
    const long long head_base = PAGED ? (long long)j * 16 * 256 : ((long long)lv.indptr[b] * p.Hkv + j) * 256;
    const long long page_stride = (long long)p.Hkv * 16 * 256;

    // ---- query fragments (B operand): column = this lane's row, k-slot = channels 16 s + 8 h
    bf16x8 qf[8];
    const int rr = row0 + wave * 32 + col;
    const bool row_ok = rr < rows_b;
    const long long out_row = (long long)(s0 + (row_ok ? rr : 0) / p.G) * p.Hq + j * p.G + (row_ok ? rr : 0) % p.G;
    {
        const uint4* qg = (const uint4*)p.q + out_row * kRowU4;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            uint4 v = qg[2 * s + h];
            if (!row_ok)
                v = make_uint4(0, 0, 0, 0);
            qf[s] = as_bf16x8(v);
        }
    }

    // ---- global -> LDS copies -------------------------------------------------------------------
    // A tile takes 16 copy instructions (8 for K, 8 for V), each covering 4 token rows.  The first half of
    // the wavefronts copies K, the other half V: wavefront w of its half issues instructions
    // w kIPW .. w kIPW + kIPW - 1.  Lane (r, c) of instruction q fetches piece c ^ swz(row) of row 4 q + r.
    // Rows past the end of the split are clamped to its last token (their scores are masked later).
    // A wavefront's rows of a tile lie in one page, so the page number is uniform over it.
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;
    const int lane_row = lane >> 4;
    const bool copies_v = wave >= WAVES / 2;
    const int row_first = 4 * kIPW * (copies_v ? wave - WAVES / 2 : wave);  // of this wavefront's rows within a tile
    unsigned lane_off[kIPW];  // byte offset of this lane's piece for a full tile, relative to the tile's first row
#pragma unroll
    for (int i = 0; i < kIPW; ++i) {
        const int tl = row_first + 4 * i + lane_row;
        lane_off[i] = (unsigned)((4 * i + lane_row) * (unsigned)tok_stride + (((lane & 15) ^ swz(tl)) << 4));
    }
    const char* const tensor = copies_v ? vg : kg;
    const char* const first_row = tensor + head_base + (long long)row_first * tok_stride;  // contiguous KV: + tile's first token
    uint4* const ring_lds = lds + ((copies_v ? kRing * kTileBytes : 0) + row_first * 256) / 16;
    // page number of the next tile to be copied, fetched one tile ahead of its use
    int next_page = 0;
    auto fetch_page = [&](int tile) __attribute__((always_inline)) {
        if (PAGED)
            next_page = pages[min(t0 + tile * kTileN + row_first, t1 - 1) >> 4];
    };
    fetch_page(0);
    auto issue_tile = [&](int tile) __attribute__((always_inline)) {
        const int tb = t0 + tile * kTileN;
        uint4* const dst = ring_lds + (tile % kRing) * (kTileBytes / 16);
        const bool full = tb + kTileN <= t1;
        const int tg = min(tb + row_first, t1 - 1);  // this wavefront's first row, clamped
        const char* const src = PAGED ? tensor + (long long)next_page * page_stride + head_base + (tg & 15) * 256
                                      : first_row + (long long)(full ? tb : tg - row_first) * tok_stride;
#pragma unroll
        for (int i = 0; i < kIPW; ++i) {
            unsigned off = lane_off[i];
            if (!full) {
                const int row = min(tg + 4 * i + lane_row, t1 - 1) - tg;  // clamped row, relative to the first
                off = (unsigned)(row * (unsigned)tok_stride + (((lane & 15) ^ swz(row_first + 4 * i + lane_row)) << 4));
            }
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + off),
                                             (__attribute__((address_space(3))) void*)(dst + i * 64), 16, 0, 0);
        }
        fetch_page(tile + 1);
    };

    // ---- per-lane LDS addresses of the MFMA operand fragments (relative to a tile) ---------------
    // K fragment st: row col, piece (2 st + h) ^ swz(col).  2 st has no bit 0 and h is bit 0 only, so the
    // piece is 2 st ^ (h ^ swz(col)) and its byte offset 32 st ^ k_xor.
    const unsigned k_row = (unsigned)(col * 256), k_xor = (unsigned)((h ^ swz(col)) << 4);
    // V fragment (ks, db), half `part`: source lane (r, q4) of a 16-lane group points at token
    // 16 ks + 8 part + 4 h + r, channels 32 db + 16 g16 + 4 q4 .. + 3; the transposing read then
    // hands lane i of the group the four tokens of channel 32 db + 16 g16 + i.  The token step
    // 16 ks only adds 4096 ks bytes (swz is periodic in 16) and goes into the offset field.
    unsigned v_off[4][2];
    {
        const int g16 = (lane >> 4) & 1, r = (lane & 15) >> 2, q4 = lane & 3;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int part = 0; part < 2; ++part) {
                const int tok = 8 * part + 4 * h + r;
                const int piece = 4 * db + 2 * g16 + (q4 >> 1);
                v_off[db][part] = (unsigned)(tok * 256 + ((piece ^ swz(tok)) << 4) + (q4 & 1) * 8);
            }
    }

    float m_run = -INFINITY, l_run = 0.f;
    floatx16 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            o[db][i] = 0.f;

    // One MFMA region: the scores of the tile in K slot `kstage` into `sn` (8 MFMAs), alternating
    // with O^T += V^T P^T for the tile in V slot `vstage` and probabilities `pp` (8 more), and between the
    // MFMAs the probabilities `pn` of the scores `so` of the tile before (their sum over the lane is
    // returned).  The three work on different tiles and do not depend on each other, so the
    // accumulator chains hide each other's latency and the vector instructions issue in the MFMAs'
    // shadow: a wavefront alone on its SIMD otherwise leaves the matrix cores idle during the
    // softmax and the vector ALU idle during the products.  Fragments are read kAhead ahead of
    // their MFMA.
    // Ring of fragment registers: kAhead + 1 reads in flight, and one more slot so that a new
    // read never targets the registers of the MFMA issued just before it.
    // A K fragment is one 128-bit read into `ring`; a V fragment is two 64-bit reads into
    // `ring_lo` / `ring_hi`, put together only after the wait that precedes its MFMA (the wait
    // names all of them as operands, so nothing that reads a fragment register can be placed
    // before the data has arrived).  What remains an assumption is that the compiler neither copies
    // nor spills a fragment register between its read and that wait; the kernels built from this
    // body use no scratch memory, and a host-side test of the build keeps it that way.
    u32x4 ring[kAhead + 2];
    u32x2 ring_lo[kAhead + 2], ring_hi[kAhead + 2];
    auto region = [&](auto qk_tag, auto sm_tag, auto pv_tag, int kstage, int vstage, floatx16& sn, const floatx16& so,
                      bf16x8 (&pn)[2], const bf16x8 (&pp)[2]) __attribute__((always_inline)) -> float {
        constexpr bool QK = decltype(qk_tag)::value, SM = decltype(sm_tag)::value, PV = decltype(pv_tag)::value;
        constexpr int NF = frag_count<QK, PV>();
        // (opaque to the optimiser, which would otherwise keep a running address per fragment)
        unsigned kbase = lds_base + (unsigned)kstage * kTileBytes;
        unsigned vbase = lds_base + (unsigned)(kRing + vstage) * kTileBytes;
        asm("" : "+s"(kbase), "+s"(vbase));
        if (QK) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                sn[i] = 0.f;
        }
        auto issue = [&](auto kc) __attribute__((always_inline)) {
            constexpr int K = decltype(kc)::value;
            if constexpr (K < NF) {
                using F = Frag<QK, PV, K>;
                if constexpr (!F::is_pv) {
                    const unsigned addr = kbase + k_row + ((32u * F::a) ^ k_xor);
                    u32x4& dst = ring[K % (kAhead + 2)];
                    asm volatile("ds_read_b128 %0, %1" : "=v"(dst) : "v"(addr));
                } else {
                    u32x2& lo = ring_lo[K % (kAhead + 2)];
                    u32x2& hi = ring_hi[K % (kAhead + 2)];
                    const unsigned a0 = vbase + v_off[F::b][0], a1 = vbase + v_off[F::b][1];
                    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%4\n\tds_read_b64_tr_b16 %1, %3 offset:%4"
                                 : "=&v"(lo), "=&v"(hi)
                                 : "v"(a0), "v"(a1), "n"(F::a * 4096));
                }
            }
        };
        auto consume = [&](auto kc) __attribute__((always_inline)) {
            constexpr int K = decltype(kc)::value;
            using F = Frag<QK, PV, K>;
            if constexpr (!F::is_pv) {
                u32x4& f = ring[K % (kAhead + 2)];
                asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(f) : "n"(ops_after<QK, PV, K>()));
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f), qf[F::a], sn, 0, 0, 0);
            } else {
                u32x2& lo = ring_lo[K % (kAhead + 2)];
                u32x2& hi = ring_hi[K % (kAhead + 2)];
                asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(lo), "+v"(hi) : "n"(ops_after<QK, PV, K>()));
                const u32x4 f = {lo[0], lo[1], hi[0], hi[1]};
                o[F::b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f), pp[F::a], o[F::b], 0, 0, 0);
            }
        };
        // Slot e of the softmax: the exponent of score e, the exponential of score e - 1, the sum of score
        // e - 2 (three short chains side by side, none waiting for the one before it).
        float psum = 0.f, x[16], pv[16];
        uint32_t w[8];
        auto soft = [&](auto ec) __attribute__((always_inline)) {
            constexpr int e = decltype(ec)::value;
            if constexpr (SM && e >= 0 && e < 18) {
                if constexpr (e < 16)
                    x[e] = __builtin_fmaf(so[e], p.scale_log2, -m_run);
                if constexpr (e >= 1 && e < 17)
                    pv[e - 1] = __builtin_amdgcn_exp2f(x[e - 1]);
                if constexpr (e >= 2) {
                    psum += pv[e - 2];
                    if constexpr ((e & 1) != 0)
                        w[(e - 2) >> 1] = pack_bf16_rne(pv[e - 3], pv[e - 2]);
                }
            }
        };
        for_each_index(issue, std::make_integer_sequence<int, kAhead + 1>{});
        // the first slots pass while the first fragments are under way
        constexpr int kLead = 18 - NF > 0 ? 18 - NF : 0;
        if constexpr (SM) {
            for_each_index(soft, std::make_integer_sequence<int, kLead>{});
            __builtin_amdgcn_sched_barrier(0);
        }
        for_each_index(
            [&](auto kc) __attribute__((always_inline)) {
                consume(kc);
                issue(std::integral_constant<int, decltype(kc)::value + kAhead + 1>{});
                if constexpr (SM) {
                    soft(std::integral_constant<int, decltype(kc)::value + kLead>{});
                    __builtin_amdgcn_sched_barrier(0);
                }
            },
            std::make_integer_sequence<int, NF>{});
        if constexpr (SM) {
            static_assert(kLead + NF >= 18, "every score gets its slot");
            const uint4 p0 = make_uint4(w[0], w[1], w[2], w[3]), p1 = make_uint4(w[4], w[5], w[6], w[7]);
            pn[0] = as_bf16x8(p0);
            pn[1] = as_bf16x8(p1);
        }
        return psum;
    };

    // The scores of tiles 0 and 1 together (two independent accumulator chains).
    auto first_scores = [&](floatx16& s0, floatx16& s1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            s0[i] = s1[i] = 0.f;
        auto issue = [&](auto kc) __attribute__((always_inline)) {
            constexpr int K = decltype(kc)::value;
            if constexpr (K < 16) {
                const unsigned addr = lds_base + (K & 1) * kTileBytes + k_row + ((32u * (K >> 1)) ^ k_xor);
                u32x4& dst = ring[K % (kAhead + 2)];
                asm volatile("ds_read_b128 %0, %1" : "=v"(dst) : "v"(addr));
            }
        };
        for_each_index(issue, std::make_integer_sequence<int, kAhead + 1>{});
        for_each_index(
            [&](auto kc) __attribute__((always_inline)) {
                constexpr int K = decltype(kc)::value, kAfter = K + kAhead < 16 ? kAhead : 15 - K;
                u32x4& f = ring[K % (kAhead + 2)];
                asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(f) : "n"(kAfter));
                floatx16& sc = (K & 1) ? s1 : s0;
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(f), qf[K >> 1], sc, 0, 0, 0);
                issue(std::integral_constant<int, K + kAhead + 1>{});
            },
            std::make_integer_sequence<int, 16>{});
    };

    // Online softmax: (m, l) of the row and the probabilities of a tile.  Scores stay unscaled in the
    // accumulator; the scale is folded into the exponent: p = 2^(s * scale - m).
    auto mask_tile = [&](int tb, floatx16& sc) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            // accumulator register i of lane-half h is token 8 (i/4) + 4 h + i%4
            const int t = tb + 8 * (i >> 2) + 4 * h + (i & 3);
            if (t >= t1)
                sc[i] = -INFINITY;
        }
    };
    auto probabilities = [&](const floatx16& sc, bf16x8 (&pn)[2]) __attribute__((always_inline)) -> float {
        float psum = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[8 * u + e], p.scale_log2, -m_run));
                psum += pv[e];
            }
            uint4 pu;
            pu.x = pack_bf16_rne(pv[0], pv[1]);
            pu.y = pack_bf16_rne(pv[2], pv[3]);
            pu.z = pack_bf16_rne(pv[4], pv[5]);
            pu.w = pack_bf16_rne(pv[6], pv[7]);
            pn[u] = as_bf16x8(pu);
        }
        return psum;
    };
    // The reference maximum m only has to bound the exponents.  After the first tile it is looked at
    // again only when a lane's 16 probabilities add up to more than kRaise (none of them is above
    // that otherwise: exact in fp32 and bf16 alike), so that most tiles find no maximum, exchange
    // nothing between lanes and rescale nothing.
    constexpr float kRaise = 1024.f;
    auto raise_maximum = [&](const floatx16& sc) __attribute__((always_inline)) -> float {
        float tmax = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i)
            tmax = fmaxf(tmax, sc[i]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32)) * p.scale_log2;
        const float m_up = fmaxf(m_run, tmax);
        const float corr = __builtin_amdgcn_exp2f(m_run - m_up);
        m_run = m_up;
        return corr;
    };
    // Takes in a tile's sum of probabilities; raises the maximum, and does the tile's probabilities again,
    // if it has to.  O holds every earlier tile by then.
    auto take_sum = [&](float psum, const floatx16& sc, bf16x8 (&pn)[2]) __attribute__((always_inline)) {
        if (__ballot(!(psum <= kRaise)) != 0) {
            const float corr = raise_maximum(sc);
            psum = probabilities(sc, pn);
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    o[db][i] *= corr;
        }
        l_run += psum;
    };

    // ---- pipeline over tiles ----------------------------------------------------------------------
    // Step t computes the scores of tile t, the probabilities of tile t-1 and P V of tile t-2 in one MFMA
    // region.  It starts the copies of K of tile t + A and V of tile t + A - 2 (A = kCopyAhead; both are
    // A steps ahead of their use, 64 KB per workgroup under way), then runs the region, waits until its
    // own copies of K of tile t+1 and V of tile t-1 have landed, and meets the other wavefronts at a
    // barrier.  A copy into a ring slot is issued only after a barrier that every wavefront reaches
    // after its last read of that slot, and a tile is read only after a barrier that every
    // wavefront reaches after its copies of that tile landed.
    const int ntiles = (t1 - t0 + kTileN - 1) / kTileN;
    const std::true_type yes{};
    const std::false_type no{};
    auto start_copies = [&](int t) __attribute__((always_inline)) {
        const int tile = copies_v ? t + kCopyAhead - 2 : t + kCopyAhead;
        if (tile >= 0 && tile < ntiles)
            issue_tile(tile);
    };
    // Waits until at most `tiles` later tiles of this wavefront's copies are under way; everybody has then.
    auto wait_copies = [&](int tiles) __attribute__((always_inline)) {
        if (tiles >= kCopyAhead - 1)
            wait_vmcnt<(kCopyAhead - 1) * kIPW>();
        else if (tiles == 2)
            wait_vmcnt<2 * kIPW>();
        else if (tiles == 1)
            wait_vmcnt<kIPW>();
        else
            wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
    };
    static_assert(kCopyAhead == 4, "wait_copies lists the counts below kCopyAhead - 1");
    // At the end of step t the copies of up to A - 1 later tiles may be under way (fewer near the end; the
    // count is that of the K copies, V has more; after the last step everything has landed).
    auto end_of_step = [&](int t) __attribute__((always_inline)) { wait_copies(ntiles - 2 - t); };
    floatx16 sa, sb;      // scores of tiles with an even / odd number
    bf16x8 pa[2], pb[2];  // their probabilities, B-operand layout
#pragma unroll
    for (int t = -kCopyAhead; t <= 0; ++t)  // K of tiles 0 .. A, V of tiles 0 .. A-2
        start_copies(t);
    end_of_step(0);
    if (ntiles > 1) {
        // steps 0 and 1 in one; the copies of step 1 wait until the slots of K of tiles 0 and 1 are free
        first_scores(sa, sb);
        // the first reference is the maximum of 64 tokens (tile 0 is whole; where tile 1 is not, the rows
        // past its end repeat its last token)
        raise_maximum(sa);
        raise_maximum(sb);
        l_run = probabilities(sa, pa);
        wait_copies(min(ntiles - 3, kCopyAhead - 2));
        start_copies(1);
        // two steps a round, so that scores and probabilities change roles instead of registers
        int t = 2;
        for (; t + 1 < ntiles; t += 2) {
            start_copies(t);
            take_sum(region(yes, yes, yes, t % kRing, (t - 2) % kRing, sa, sb, pb, pa), sb, pb);
            end_of_step(t);
            start_copies(t + 1);
            take_sum(region(yes, yes, yes, (t + 1) % kRing, (t - 1) % kRing, sb, sa, pa, pb), sa, pa);
            end_of_step(t + 1);
        }
        if (t < ntiles) {
            start_copies(t);
            take_sum(region(yes, yes, yes, t % kRing, (t - 2) % kRing, sa, sb, pb, pa), sb, pb);
            end_of_step(t);
            sb = sa;  // the last tile's scores
            pa[0] = pb[0];  // and the probabilities of the one before
            pa[1] = pb[1];
        }
        // the last tile; only it can be ragged
        if (t0 + ntiles * kTileN > t1)
            mask_tile(t0 + (ntiles - 1) * kTileN, sb);
        take_sum(region(no, yes, yes, 0, (ntiles - 2) % kRing, sa, sb, pb, pa), sb, pb);
    } else {
        region(yes, no, no, 0, 0, sa, sa, pa, pa);
        mask_tile(t0, sa);
        raise_maximum(sa);
        l_run = probabilities(sa, pb);
    }
    region(no, no, yes, 0, (ntiles - 1) % kRing, sa, sa, pa, pb);

    // ---- write the partial state ------------------------------------------------------------------
    const float l = l_run + __shfl_xor(l_run, 32);
    if (!row_ok)
        return;
    const long long prow = part_index(p, out_row, lv.slot0 + split);
    if (h == 0)
        p.part_ml[prow] = make_float2(m_run, l);
    // the split's own normalised output, fp16 (l > 0: a split holds at least one token)
    const float inv_l = 1.f / l;
    __half* dst = (__half*)p.part_acc + prow * kD;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            // registers 4 q4 .. 4 q4 + 3 are channels 32 db + 8 q4 + 4 h .. + 3
            const __half2 lo = __floats2half2_rn(o[db][4 * q4] * inv_l, o[db][4 * q4 + 1] * inv_l);
            const __half2 hi = __floats2half2_rn(o[db][4 * q4 + 2] * inv_l, o[db][4 * q4 + 3] * inv_l);
            uint2 v;
            v.x = *reinterpret_cast<const uint32_t*>(&lo);
            v.y = *reinterpret_cast<const uint32_t*>(&hi);
            *reinterpret_cast<uint2*>(dst + 32 * db + 8 * q4 + 4 * h) = v;
        }
}

}  // namespace prefix_impl
}  // namespace spd
