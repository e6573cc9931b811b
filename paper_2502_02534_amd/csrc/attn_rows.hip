// Partial softmax states of the shapes outside the bf16 / head_dim 128 kernels: fp32 inputs, other head
// dimensions (multiples of 8 up to 256), more than 16 query heads per KV head.
//
// A work item is a block of 16 or 32 query rows of one KV head and one token range (a prefix split,
// where the rows are all samples' heads of a prompt, or a suffix chunk, where they are the heads of
// one sample).  One wavefront walks the range a tile at a time, or, where that would leave SIMDs
// idle, two or four wavefronts of a workgroup take its tiles in turn and put their states together in
// LDS at the end (more wavefronts without more partial states for the merge).
// Both products run on the matrix cores, and the operand layouts are chosen so that nothing is
// transposed on the way in:
//
//   S^T = K Q^T   A = K rows, loaded 16 bytes per lane: lane (c, r) takes token c and the channels
//                 of contraction slot r (any fixed assignment of channels to slots will do, as long
//                 as Q uses the same one); B = the query rows, held in registers
//   O  += P V     the accumulator of S^T gives lane (c, r) the scores of query c and tokens 4 r + i,
//                 which is the A operand of P with tokens 4 r + i in contraction slot r; B = V rows
//                 4 r + i, a lane holding neighbouring channels, one per product
//
//   fp32: v_mfma_f32_16x16x4_f32, tiles of 16 tokens; nothing leaves fp32.
//   bf16: v_mfma_f32_16x16x32_bf16, tiles of 32 tokens.  K and Q enter as they are (their products are
//         exact in fp32); the probabilities are fp32 and enter as the sum of three bf16 numbers of
//         eight bits each, which together are the fp32 number, i.e. three products per V fragment
//         (two leave out up to 2^-17 of a probability, which shows where values cancel; the third costs 3 %
//         of the last call below, 28.6 -> 29.6 us).
//
// Bound: HBM for the suffix chunks; for prefixes with many rows the fp32 product (32 clocks of a
// SIMD per 16x16x4 step), for a few rows latency, hence splits down to one tile per wavefront.  A
// block of 32 rows uses every loaded K and V register twice; the row blocks of one token range run
// on one XCD, whose L2 they share.
// Measured, whole call (before: one wavefront per query row, a lane per token on the vector ALU):
//   fp32, 4/1 heads of 64 channels, 4 samples, prompt 256, suffix 32           93 ->  9.4 us
//   fp32, 32/8 heads of 128 channels, 16 samples, prompt 2048, suffixes up to 256  582 ->  21 us
//   bf16, 32/8 heads of 64 channels, 3 prompts of up to 4001 tokens x 21 samples,
//   suffixes up to 501, paged                                                 840..1060 -> 25 us
// Where the last two go: launch and first loads 4 us, the tiles (from registers, 2.5 us each in fp32, 2 in bf16, with
// two to three wavefronts per SIMD: dependent products, softmax, load round trips) 10 to 15, the merge 3 (the first
// call is bound by the host).
#include "spd_internal.h"
#include "plan.h"
#include "attn_prefix_body.h"

#include <hip/hip_fp16.h>

#include <type_traits>

namespace spd {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr int kWaves = 4;  // wavefronts per workgroup (eight, sharing an item: 10 to 15 % slower)

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return *reinterpret_cast<bf16x8*>(&v); }

// Two floats to packed bf16 (round to nearest even): one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    const bf16x2 r = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<const uint32_t*>(&r);
}

// One wavefront's work: query rows row0 .. row0 + 16 QB - 1 of the `rows` rows of KV head j (row rr is
// head rr % G of sample s0 + rr / G), tokens t0 .. t1 - 1 (t0 < t1, t0 a multiple of 32) of one
// sequence, slot of the partial state.
struct RowsItem {
    const void *k, *v;
    const int* pages;   // paged KV: the sequence's page list
    long long start;    // contiguous KV: the sequence's first token
    int s0, j, row0, rows, t0, t1, slot;
    int share, part;    // wavefronts that share the item, and which of them this one is
    unsigned g_inv;     // min(floor(2^32 / G), 2^32 - 1)
};

// How K and V reach the products.
//   RING (bf16, 64 channels, long chunks: plan::rows_through_lds has the figures): tiles go from global memory straight
//     into LDS (global_load_lds_dwordx4), into two K and two V slots of the wavefront's own, two tiles ahead of their
//     use, so that a wavefront nearly alone on its SIMD does not wait for a round trip in every tile; no
//     barrier is needed.
//   otherwise: registers, reloaded in place.  (With a ring fp32 loses: 128 channels 22.3 -> 28.7 us, 128 KB of LDS
//     leave one wavefront per SIMD; 64 channels 23.7 -> 25.6, its products already hide the loads.)
constexpr int kDepth = 2;
constexpr int kRingRow = 128;              // bytes of a token row
constexpr int kRingTile = 32 * kRingRow;   // of a K or V tile
constexpr int kRingCopies = kRingTile / 1024;  // copy instructions per tile, eight rows each
// 16-byte piece p of token row `tok` lies at piece p ^ swz(tok): two rows share the 256-byte bank window, and
// the sixteen rows of a K operand get sixteen different places in it.
__device__ __forceinline__ int swz(int tok) { return (tok >> 1) & 7; }

// LDS of a wavefront: its ring, then, where several wavefronts share an item, its state.
template <int DT, int QB, bool RING> union WaveLds {
    uint4 ring[RING ? 2 * kDepth * kRingTile / 16 : 1];
    struct {
        float o[16 * QB][DT];
        float2 ml[16 * QB];
    } state;
};

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// LDS reads that the copies under way do not hold up: the compiler would wait for every copy before any
// read of its own.  Complete when they return.
// K of a tile: two places of a row (channels 0 .. 31, 32 .. 63), in the first and in the second 16 tokens.
__device__ __forceinline__ void ring_read_k(unsigned a0, unsigned a1, u32x4 (&v)[4])
{
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %4 offset:%6\n\t"
                 "ds_read_b128 %3, %5 offset:%6\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                 : "v"(a0), "v"(a1), "n"(16 * kRingRow)
                 : "memory");
}
// V of a tile: eight bytes of rows 4 i and 16 + 4 i from a[i] on.
__device__ __forceinline__ void ring_read_v(const unsigned (&a)[4], u32x2 (&v)[8])
{
    constexpr int S = 4 * kRingRow, B = 16 * kRingRow;
    asm volatile("ds_read_b64 %0, %8\n\tds_read_b64 %1, %9 offset:%12\n\t"
                 "ds_read_b64 %2, %10 offset:%13\n\tds_read_b64 %3, %11 offset:%14\n\t"
                 "ds_read_b64 %4, %8 offset:%15\n\tds_read_b64 %5, %9 offset:%16\n\t"
                 "ds_read_b64 %6, %10 offset:%17\n\tds_read_b64 %7, %11 offset:%18\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(S), "n"(2 * S), "n"(3 * S), "n"(B), "n"(B + S),
                   "n"(B + 2 * S), "n"(B + 3 * S)
                 : "memory");
}
template <int N> __device__ __forceinline__ void wait_copies()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Output row (sample, query head) of query row rr of an item.
__device__ __forceinline__ long long item_out_row(const AttnParams& p, const RowsItem& it, int rr)
{
    // rr / G: the product with the rounded-down reciprocal is the quotient or one less
    int n = (int)__umulhi((unsigned)rr, it.g_inv), g = rr - n * p.G;
    const bool low = g >= p.G;
    n += low ? 1 : 0;
    g -= low ? p.G : 0;
    return (long long)(it.s0 + n) * p.Hq + (long long)it.j * p.G + g;
}

// Stores N (4 or 8) channels of a normalised partial output.
template <typename T, int N>
__device__ __forceinline__ void store_part(const AttnParams& p, long long at, const float (&y)[N])
{
    if constexpr (std::is_same<T, float>::value) {
        *reinterpret_cast<float4*>((float*)p.part_acc + at) = make_float4(y[0], y[1], y[2], y[3]);
    } else {
        uint32_t w[N / 2];
#pragma unroll
        for (int e = 0; e < N / 2; ++e) {
            const __half2 h2 = __floats2half2_rn(y[2 * e], y[2 * e + 1]);
            w[e] = *reinterpret_cast<const uint32_t*>(&h2);
        }
        __half* dst = (__half*)p.part_acc + at;
        if constexpr (N == 8)
            *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
        else
            *reinterpret_cast<uint2*>(dst) = make_uint2(w[0], w[1]);
    }
}

// T: float or uint16_t (bf16 bits).  DT: head_dim rounded up to 64, 128 or 256; channels from p.D on are
// zero.  QB: 16-row blocks per wavefront.
template <typename T, int DT, int QB, bool PAGED, bool RING, typename Lds>
__device__ __forceinline__ void rows_body(const AttnParams& p, const RowsItem& it, Lds* lds)
{
    constexpr bool F32 = std::is_same<T, float>::value;
    constexpr int kTile = F32 ? 16 : 32;          // tokens per tile
    constexpr int kBlk = kTile / 16;              // 16-token blocks per tile
    constexpr int kEltBytes = (int)sizeof(T);
    constexpr int kKRegs = DT * kEltBytes / 64;   // 16-byte pieces of K per lane and 16-token block
    constexpr int kQRegs = kKRegs;                // 16-byte pieces of Q per lane and row block
    constexpr int kVTok = 4 * kBlk;               // V tokens per lane and tile
    constexpr int kVPiece = F32 ? 4 : (DT == 64 ? 4 : 8);  // neighbouring channels of a lane's V load
    constexpr int kVLoads = DT / (16 * kVPiece);  // V loads per token
    constexpr int kVDw = kVPiece * kEltBytes / 4; // dwords per V load
    constexpr int kCols = DT / 16;                // PV products per tile (columns c of product i: one channel each)

    const int lane = threadIdx.x & 63;
    const int r = lane >> 4, c = lane & 15;
    const int D = p.D;
    const bool padded = !RING && D != DT;
    // Token of a 16-token block that row m of the scores stands for.  (From LDS: lane-rows 0 and 1 read V rows
    // of different parity, which lie in different halves of the bank window.)
    auto token_of = [](int m) { return RING ? 4 * (m & 3) + (m >> 2) : m; };

    // ---- query rows: contraction slot r of step s holds, fp32, channels 16 s + 4 r + e (e = one product
    // each), bf16, channels 32 s + 8 r .. + 7
    auto out_row = [&](int rr) -> long long { return item_out_row(p, it, rr); };
    constexpr int kChanPerPiece = 16 / kEltBytes;
    uint4 q[QB][kQRegs];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        const int rr = it.row0 + 16 * b + c;
        const bool ok = rr < it.rows;
        const T* qp = (const T*)p.q + out_row(ok ? rr : 0) * D;
#pragma unroll
        for (int s = 0; s < kQRegs; ++s) {
            const int ch = (4 * s + r) * kChanPerPiece;
            q[b][s] = make_uint4(0u, 0u, 0u, 0u);
            if (ok && ch < D)
                q[b][s] = *reinterpret_cast<const uint4*>(qp + ch);
        }
    }

    // ---- tiles ----
    const unsigned row_elems = PAGED ? (unsigned)D : (unsigned)(p.Hkv * D);  // from one token of the head to the next
    const int last_page = PAGED ? (it.t1 - 1) >> 4 : 0;
    typedef const __attribute__((address_space(4))) int* const_int_ptr;
    const const_int_ptr pages = (const_int_ptr)it.pages;  // (uniform places: scalar loads)
    struct Base {
        long long a, b;  // element offset of the tile's first row in each of its 16-token blocks
    };
    auto tile_base = [&](int tb) -> Base {
        Base x = {0, 0};
        if (PAGED) {
            const long long pa = pages[min(tb >> 4, last_page)];
            x.a = (pa * p.Hkv + it.j) * 16 * D;
            if (kBlk == 2) {
                const long long pb = pages[min((tb >> 4) + 1, last_page)];
                x.b = (pb * p.Hkv + it.j) * 16 * D;
            }
        } else {
            x.a = ((it.start + tb) * p.Hkv + it.j) * D;
            x.b = x.a + 16ll * p.Hkv * D;
        }
        return x;
    };
    // A whole tile is loaded from its blocks' first rows plus lane offsets fixed for the range; in the
    // ragged last one tokens past the end are clamped to the last (their scores are masked).
    const unsigned koff = (unsigned)c * row_elems, voff = (unsigned)(4 * r) * row_elems;
    auto block_row = [&](int tb, const Base& base, int blk, int i, long long& first) __attribute__((always_inline)) -> unsigned {
        const int last = it.t1 - 1 - tb;           // the tile's last valid token (uniform, >= 0)
        const bool here = last >= 16 * blk;        // this block holds valid tokens
        first = blk == 0 || !here ? base.a : base.b;
        return (unsigned)(here ? min(i, last - 16 * blk) : last) * row_elems;
    };
    uint4 kk[kBlk][kKRegs];
    uint32_t vv[kVTok][kVLoads * kVDw];
    auto load_k_from = [&](int blk, const T* kp, unsigned row) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kKRegs; ++s) {
            const int ch = (4 * s + r) * kChanPerPiece;
            kk[blk][s] = *reinterpret_cast<const uint4*>(kp + (row + (unsigned)(padded && ch >= D ? 0 : ch)));
        }
    };
    auto load_v_from = [&](int t, const T* vp, unsigned row) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < kVLoads; ++g) {
            const int ch = 16 * kVPiece * g + kVPiece * c;
            const T* src = vp + (row + (unsigned)(padded && ch >= D ? 0 : ch));
            uint32_t* dst = &vv[t][g * kVDw];
            if constexpr (kVDw == 4) {
                const uint4 x = *reinterpret_cast<const uint4*>(src);
                dst[0] = x.x;
                dst[1] = x.y;
                dst[2] = x.z;
                dst[3] = x.w;
            } else {
                const uint2 x = *reinterpret_cast<const uint2*>(src);
                dst[0] = x.x;
                dst[1] = x.y;
            }
        }
    };
    // ---- ring: copies, and reads into the same registers ----
    static_assert(!RING || (!F32 && DT == 64), "the ring's layout is that of 128-byte rows and 32-token tiles");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint4* const ring = lds[wave].ring;
    const unsigned ring_at = (unsigned)(size_t)(__attribute__((address_space(3))) void*)ring;
    // Copy i brings rows 8 i .. 8 i + 7, lane L the place L % 8 of row 8 i + L / 8.  K in slots 0 .. kDepth - 1, V
    // behind them.
    auto copy_tile = [&](bool is_v, int slot, int tb, const Base& base) __attribute__((always_inline)) {
        const T* const src = (const T*)(is_v ? it.v : it.k);
        uint4* const dst = ring + ((is_v ? kDepth : 0) + slot) * (kRingTile / 16);
        const int last = it.t1 - 1 - tb;  // the tile's last valid token
#pragma unroll
        for (int i = 0; i < kRingCopies; ++i) {
            const int row = 8 * i + (lane >> 3), valid = min(row, last);  // tokens past the end are clamped to the last
            const T* at = src + (valid < 16 ? base.a : base.b) + (unsigned)(valid & 15) * row_elems + ((lane & 7) ^ swz(row)) * 8;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)at,
                                             (__attribute__((address_space(3))) void*)(dst + i * 64), 16, 0, 0);
        }
    };
    const unsigned k_at = ring_at + (unsigned)(token_of(c) * kRingRow), k_xor = (unsigned)((r ^ swz(token_of(c))) << 4);
    // (V row 4 i + r of a block: its swizzle is that of row r with the bits of 2 i flipped)
    const unsigned v_at = ring_at + (unsigned)(kDepth * kRingTile + r * kRingRow + 8 * (c & 1));
    const unsigned v_xor = (unsigned)(((c >> 1) ^ swz(r)) << 4);
    auto read_k = [&](int slot) __attribute__((always_inline)) {
        if constexpr (RING) {
            const unsigned at = k_at + (unsigned)(slot * kRingTile);
            u32x4 v[4];
            ring_read_k(at + k_xor, at + (k_xor ^ 64u), v);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                kk[i >> 1][i & 1] = make_uint4(v[i][0], v[i][1], v[i][2], v[i][3]);
        }
    };
    auto read_v = [&](int slot) __attribute__((always_inline)) {
        if constexpr (RING) {
            unsigned a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                a[i] = v_at + (unsigned)(slot * kRingTile) + (v_xor ^ (32u * (unsigned)i));
            u32x2 v[8];
            ring_read_v(a, v);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                vv[t][0] = v[t][0];
                vv[t][1] = v[t][1];
            }
        }
    };
    auto load_k = [&](int tb, const Base& base) __attribute__((always_inline)) {
        if (tb + kTile <= it.t1) {
#pragma unroll
            for (int blk = 0; blk < kBlk; ++blk)
                load_k_from(blk, (const T*)it.k + (blk == 0 ? base.a : base.b), koff);
        } else {
#pragma unroll
            for (int blk = 0; blk < kBlk; ++blk) {
                long long first;
                const unsigned row = block_row(tb, base, blk, c, first);
                load_k_from(blk, (const T*)it.k + first, row);
            }
        }
    };
    auto load_v = [&](int tb, const Base& base) __attribute__((always_inline)) {
        if (tb + kTile <= it.t1) {
#pragma unroll
            for (int t = 0; t < kVTok; ++t)
                load_v_from(t, (const T*)it.v + (t < 4 ? base.a : base.b) + (size_t)(t & 3) * row_elems, voff);
        } else {
#pragma unroll
            for (int t = 0; t < kVTok; ++t) {
                long long first;
                const unsigned row = block_row(tb, base, t >> 2, 4 * r + (t & 3), first);
                load_v_from(t, (const T*)it.v + first, row);
            }
        }
    };

    float m_run[QB], l_run[QB];  // of query row c of each block; l_run: this lane's share
    floatx4 o[QB][kCols];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        m_run[b] = -INFINITY;
        l_run[b] = 0.f;
#pragma unroll
        for (int i = 0; i < kCols; ++i)
            o[b][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    // K is reloaded in place as soon as the scores have read it, V after P V: one set of registers
    // leaves room for two or more wavefronts per SIMD up to 128 channels, whose phases cover each other's
    // loads (for one with more).
    const int tfirst = it.t0 + it.part * kTile, tstep = it.share * kTile;
    const int tlast = (it.t1 - 1) & ~(kTile - 1);  // the range's last tile
    constexpr int kAhead = RING ? kDepth : 1;  // tiles between a load and its use
    if (tfirst < it.t1) {
        const Base base = tile_base(tfirst);
        if constexpr (RING) {
            copy_tile(false, 0, tfirst, base);
            copy_tile(true, 0, tfirst, base);
            if (tfirst + tstep < it.t1) {
                const Base second = tile_base(tfirst + tstep);
                copy_tile(false, 1, tfirst + tstep, second);
                copy_tile(true, 1, tfirst + tstep, second);
            }
        } else {
            load_k(tfirst, base);
            load_v(tfirst, base);
        }
    }
    static_assert(kDepth == 2, "two tiles are copied ahead of the loop, and the waits count on it");
    Base next_base = tile_base(min(tfirst + kAhead * tstep, tlast));
    int slot = 0;
    for (int tb = tfirst; tb < it.t1; tb += tstep) {
        const bool more = tb + kAhead * tstep < it.t1;
        const Base base = next_base;  // of the tile kAhead tiles on
        if constexpr (RING) {
            // copies after K of this tile: V of it, K and V of the next (the last tile: its V)
            if (tb + tstep < it.t1)
                wait_copies<3 * kRingCopies>();
            else
                wait_copies<kRingCopies>();
            read_k(slot);
            if (more)
                copy_tile(false, slot, tb + kAhead * tstep, base);
        }
        if (padded) {  // channels past the head dimension
#pragma unroll
            for (int blk = 0; blk < kBlk; ++blk)
#pragma unroll
                for (int s = 0; s < kKRegs; ++s)
                    if ((4 * s + r) * kChanPerPiece >= D)
                        kk[blk][s] = make_uint4(0u, 0u, 0u, 0u);
        }
        // ---- scores: lane (c, r), register i of block blk = token tb + 16 blk + 4 r + i for query c
        floatx4 sacc[QB][kBlk];
#pragma unroll
        for (int b = 0; b < QB; ++b)
#pragma unroll
            for (int blk = 0; blk < kBlk; ++blk)
                sacc[b][blk] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kKRegs; ++s)
#pragma unroll
            for (int blk = 0; blk < kBlk; ++blk)
#pragma unroll
                for (int b = 0; b < QB; ++b) {
                    const uint4 a = kk[blk][s], w = q[b][s];
                    if constexpr (F32) {
                        sacc[b][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(w.x), sacc[b][blk], 0, 0, 0);
                        sacc[b][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(w.y), sacc[b][blk], 0, 0, 0);
                        sacc[b][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(w.z), sacc[b][blk], 0, 0, 0);
                        sacc[b][blk] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(w.w), sacc[b][blk], 0, 0, 0);
                    } else {
                        sacc[b][blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(w), sacc[b][blk], 0, 0, 0);
                    }
                }
        if (more) {
            if constexpr (!RING)
                load_k(tb + tstep, base);
            next_base = tile_base(min(tb + (kAhead + 1) * tstep, tlast));
        }
        // ---- online softmax, base 2.  The reference maximum only has to bound the exponents: after the first
        // tile it is looked at again only when a lane's probabilities add up to more than kRaise
        // (none of them is above that otherwise), or while a query has met no score but -inf (such tiles
        // add nothing); most tiles then exchange nothing between lanes and rescale nothing.
        constexpr float kRaise = 1024.f;
        float pv[QB][kVTok];
#pragma unroll
        for (int b = 0; b < QB; ++b) {
            float sc[kVTok];
#pragma unroll
            for (int t = 0; t < kVTok; ++t)
                sc[t] = sacc[b][t >> 2][t & 3];
            if (tb + kTile > it.t1) {  // only the last tile of a range can be ragged
#pragma unroll
                for (int t = 0; t < kVTok; ++t)
                    if (tb + 16 * (t >> 2) + token_of(4 * r + (t & 3)) >= it.t1)
                        sc[t] = -INFINITY;
            }
            auto probabilities = [&](float ref) __attribute__((always_inline)) -> float {
                float psum = 0.f;
#pragma unroll
                for (int t = 0; t < kVTok; ++t) {
                    pv[b][t] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[t], p.scale_log2, -ref));
                    psum += pv[b][t];
                }
                return psum;
            };
            float psum = 0.f;
            bool raise = true;
            if (__ballot(m_run[b] == -INFINITY) == 0ull) {
                psum = probabilities(m_run[b]);
                raise = __ballot(!(psum <= kRaise)) != 0ull;
            }
            if (raise) {
                float tmax = sc[0];
#pragma unroll
                for (int t = 1; t < kVTok; ++t)
                    tmax = fmaxf(tmax, sc[t]);
                tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
                tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
                const float m_new = fmaxf(m_run[b], tmax * p.scale_log2);
                const float ref = m_new == -INFINITY ? 0.f : m_new;
                const float corr = __builtin_amdgcn_exp2f(m_run[b] - ref);
                psum = probabilities(ref);
                l_run[b] *= corr;
                m_run[b] = m_new;
                // accumulator register i of lane-row r belongs to query 4 r + i
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float f = __shfl(corr, 4 * r + i);
#pragma unroll
                    for (int k = 0; k < kCols; ++k)
                        o[b][k][i] *= f;
                }
            }
            l_run[b] += psum;
        }
        if constexpr (RING) {
            // copies after V of this tile: K and V of the next, K of the one after
            if (more)
                wait_copies<3 * kRingCopies>();
            else if (tb + tstep < it.t1)
                wait_copies<2 * kRingCopies>();
            else
                wait_copies<0>();
            read_v(slot);
            if (more)
                copy_tile(true, slot, tb + kAhead * tstep, base);
            slot ^= 1;
        }
        // ---- O += P V: column c of product k is channel kVPiece (16 (k / kVPiece) + c) + k % kVPiece
        if constexpr (F32) {
            // Past the end of the range the last token's values were loaded: zeros in their place, since
            // a probability of zero does not take an infinite value out.
            if (tb + kTile > it.t1) {
#pragma unroll
                for (int t = 0; t < kVTok; ++t)
                    if (tb + token_of(4 * r + t) >= it.t1)
#pragma unroll
                        for (int k = 0; k < kCols; ++k)
                            vv[t][k] = 0u;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < kCols; ++k)
#pragma unroll
                    for (int b = 0; b < QB; ++b)
                        o[b][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[b][i], __uint_as_float(vv[i][k]), o[b][k], 0, 0, 0);
        } else {
            uint4 term[3][QB];  // the probabilities, most significant bits first
#pragma unroll
            for (int b = 0; b < QB; ++b)
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    uint32_t w[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        w[t] = pack_bf16(pv[b][2 * t], pv[b][2 * t + 1]);
                        if (e < 2) {  // what is left (exact)
                            pv[b][2 * t] -= __uint_as_float(w[t] << 16);
                            pv[b][2 * t + 1] -= __uint_as_float(w[t] & 0xffff0000u);
                        }
                    }
                    term[e][b] = make_uint4(w[0], w[1], w[2], w[3]);
                }
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const uint32_t sel = (k & 1) ? 0x07060302u : 0x05040100u;
                uint4 f;  // V of the lane's eight tokens, one channel
                f.x = __builtin_amdgcn_perm(vv[1][k >> 1], vv[0][k >> 1], sel);
                f.y = __builtin_amdgcn_perm(vv[3][k >> 1], vv[2][k >> 1], sel);
                f.z = __builtin_amdgcn_perm(vv[5][k >> 1], vv[4][k >> 1], sel);
                f.w = __builtin_amdgcn_perm(vv[7][k >> 1], vv[6][k >> 1], sel);
#pragma unroll
                for (int e = 2; e >= 0; --e)
#pragma unroll
                    for (int b = 0; b < QB; ++b)
                        o[b][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(term[e][b]), as_bf16x8(f), o[b][k], 0, 0, 0);
            }
        }
        if (!RING && more)
            load_v(tb + tstep, base);
    }

    // ---- the partial state ----
    const bool shared = it.share > 1;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        float l = l_run[b];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int rr = it.row0 + 16 * b + c;
        if (r == 0) {
            if (shared)
                lds[wave].state.ml[16 * b + c] = make_float2(m_run[b], l);
            else if (rr < it.rows)
                p.part_ml[part_index(p, out_row(rr), it.slot)] = make_float2(m_run[b], l);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float lq = __shfl(l, 4 * r + i);
            const int row = 16 * b + 4 * r + i;
            const float inv = lq > 0.f ? 1.f / lq : 0.f;
#pragma unroll
            for (int g = 0; g < kVLoads; ++g) {
                const int ch = 16 * kVPiece * g + kVPiece * c;
                float y[kVPiece];
#pragma unroll
                for (int e = 0; e < kVPiece; ++e)
                    y[e] = o[b][kVPiece * g + e][i];
                if (shared) {
#pragma unroll
                    for (int e = 0; e < kVPiece; e += 4)
                        *reinterpret_cast<float4*>(&lds[wave].state.o[row][ch + e]) = make_float4(y[e], y[e + 1], y[e + 2], y[e + 3]);
                } else if (it.row0 + row < it.rows && !(padded && ch >= D)) {
#pragma unroll
                    for (int e = 0; e < kVPiece; ++e)
                        y[e] *= inv;
                    store_part<T, kVPiece>(p, part_index(p, out_row(it.row0 + row), it.slot) * D + ch, y);
                }
            }
        }
    }
}

// The states that the wavefronts of an item left in LDS, put together by those wavefronts (after a
// workgroup barrier) and stored.
template <typename T, int DT, int QB, typename Lds>
__device__ __forceinline__ void combine_shared(const AttnParams& p, const RowsItem& it, const Lds* lds)
{
    constexpr int kThreadsPerRow = DT / 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), w0 = wave - it.part;
    const int tid = it.part * 64 + (int)(threadIdx.x & 63);
    for (int x = tid; x < 16 * QB * kThreadsPerRow; x += it.share * 64) {
        const int row = x / kThreadsPerRow, ch = x % kThreadsPerRow * 4;
        float m = -INFINITY, l = 0.f;
        for (int w = 0; w < it.share; ++w)
            m = fmaxf(m, lds[w0 + w].state.ml[row].x);
        const float ref = m == -INFINITY ? 0.f : m;
        float y[4] = {0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < it.share; ++w) {
            const float2 ml = lds[w0 + w].state.ml[row];
            const float f = __builtin_amdgcn_exp2f(ml.x - ref);
            const float4 a = *reinterpret_cast<const float4*>(&lds[w0 + w].state.o[row][ch]);
            l = __builtin_fmaf(ml.y, f, l);
            y[0] = __builtin_fmaf(a.x, f, y[0]);
            y[1] = __builtin_fmaf(a.y, f, y[1]);
            y[2] = __builtin_fmaf(a.z, f, y[2]);
            y[3] = __builtin_fmaf(a.w, f, y[3]);
        }
        if (it.row0 + row >= it.rows)
            continue;
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            y[e] *= inv;
        const long long prow = part_index(p, item_out_row(p, it, it.row0 + row), it.slot);
        if (ch < p.D)
            store_part<T, 4>(p, prow * p.D + ch, y);
        if (ch == 0)
            p.part_ml[prow] = make_float2(m, l);
    }
}

// Marks the rows of an empty token range: l = 0 tells the merge to leave the slot out (its output
// part stays unwritten).
__device__ __forceinline__ void mark_empty(const AttnParams& p, const RowsItem& it, int count)
{
    const int lane = (int)(threadIdx.x & 63), rr = it.row0 + lane;
    if (it.part == 0 && lane < count && rr < it.rows)
        p.part_ml[part_index(p, item_out_row(p, it, rr), it.slot)] = make_float2(-INFINITY, 0.f);
}

// One item (or, with nothing to do, `live` = false): every wavefront of the workgroup calls this with
// the same `share`.
template <typename T, int DT, int QB, bool PAGED, bool RING, typename Lds>
__device__ __forceinline__ void run_item(const AttnParams& p, const RowsItem& it, bool live, Lds* lds)
{
    const bool some = live && it.t0 < it.t1;
    if (some)
        rows_body<T, DT, QB, PAGED, RING>(p, it, lds);
    else if (live)
        mark_empty(p, it, 16 * QB);
    if (it.share > 1) {
        __syncthreads();
        if (some)
            combine_shared<T, DT, QB>(p, it, lds);
    }
}

struct RowsLaunch {
    int prefix_blocks, prefix_rowblocks;  // workgroups with prefix items; row blocks per (split, prompt, KV head)
    int prefix_share, suffix_share;       // wavefronts per item (a power of two, at most a workgroup's)
    unsigned suffix_items, g_inv;
};

// Prefix and suffix items in one launch: workgroups below prefix_blocks take prefix items (the row
// blocks of one split, prompt and KV head on one XCD), the others suffix items (row block fastest, then KV
// head, so that neighbours read the heads of the same tokens, one contiguous stretch; then suffix_place's order).
template <typename T, int DT, int QB, bool PAGED, bool RING>
__global__ __launch_bounds__(kWaves * 64) void attn_rows_kernel(AttnParams p, RowsLaunch a)
{
    __shared__ WaveLds<DT, QB, RING> lds[kWaves];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    RowsItem it;
    it.g_inv = a.g_inv;
    if ((int)blockIdx.x < a.prefix_blocks) {
        it.share = a.prefix_share;
        it.part = wave & (it.share - 1);
        const int per = kWaves / it.share;  // neighbouring row blocks a workgroup takes
        const int rowtiles = (a.prefix_rowblocks + per - 1) / per;
        const prefix_impl::PrefixItem at = prefix_impl::prefix_item((int)blockIdx.x, p.num_prefix_splits, rowtiles, p.B * p.Hkv);
        const int b = at.z / p.Hkv;
        it.j = at.z % p.Hkv;
        it.s0 = p.sample_indptr[b];
        it.rows = (p.sample_indptr[b + 1] - it.s0) * p.G;
        it.row0 = (at.rowtile * per + wave / it.share) * 16 * QB;
        it.t0 = at.split * p.prefix_split_tokens;
        it.t1 = min(p.prefix_lens[b], it.t0 + p.prefix_split_tokens);
        it.slot = p.prefix_slot0 + at.split;
        it.k = p.k_prefix;
        it.v = p.v_prefix;
        it.start = PAGED ? 0 : p.prefix_indptr[b];
        it.pages = PAGED ? p.prefix_pages + p.prefix_indptr[b] : nullptr;
        run_item<T, DT, QB, PAGED, RING>(p, it, it.row0 < it.rows, lds);
    } else {
        it.share = a.suffix_share;
        it.part = wave & (it.share - 1);
        const int rowblocks = (p.G + 15) / 16;
        const unsigned item = (blockIdx.x - (unsigned)a.prefix_blocks) * (unsigned)(kWaves / it.share) + (unsigned)(wave / it.share);
        const bool live = item < a.suffix_items;
        unsigned rest = live ? item : 0u;
        it.row0 = 0;
        if (rowblocks > 1) {
            it.row0 = (int)(rest % (unsigned)rowblocks) * 16;
            rest /= (unsigned)rowblocks;
        }
        it.j = (int)(rest % (unsigned)p.Hkv);
        rest /= (unsigned)p.Hkv;
        const plan::SuffixPlace at = plan::suffix_place(rest, (unsigned)p.N);
        const int chunk = at.chunk, n = at.n;
        it.s0 = n;
        it.rows = p.G;
        it.t0 = chunk * p.suffix_chunk_tokens;
        it.t1 = min(p.suffix_lens[n], it.t0 + p.suffix_chunk_tokens);
        it.slot = p.suffix_slot0 + chunk;
        it.k = p.k_suffix;
        it.v = p.v_suffix;
        it.start = (long long)n * p.max_suffix_len;
        it.pages = PAGED ? p.suffix_pages + p.suffix_page_indptr[n] : nullptr;
        run_item<T, DT, 1, PAGED, RING>(p, it, live, lds);
    }
}

template <typename T, int DT, int QB, bool RING>
void launch_rows(const AttnParams& p, unsigned grid, const RowsLaunch& a, hipStream_t s)
{
    if (p.page_size)
        hipLaunchKernelGGL((attn_rows_kernel<T, DT, QB, true, RING>), dim3(grid), dim3(kWaves * 64), 0, s, p, a);
    else
        hipLaunchKernelGGL((attn_rows_kernel<T, DT, QB, false, RING>), dim3(grid), dim3(kWaves * 64), 0, s, p, a);
}

template <typename T>
void launch_rows_dim(const AttnParams& p, int qb, bool ring, unsigned grid, const RowsLaunch& a, hipStream_t s)
{
    constexpr bool kRing = std::is_same<T, uint16_t>::value;
    if (kRing && ring)
        qb == 1 ? launch_rows<T, 64, 1, kRing>(p, grid, a, s) : launch_rows<T, 64, 2, kRing>(p, grid, a, s);
    else if (p.D <= 64)
        qb == 1 ? launch_rows<T, 64, 1, false>(p, grid, a, s) : launch_rows<T, 64, 2, false>(p, grid, a, s);
    else if (p.D <= 128)  // (one row block: rows_per_block)
        launch_rows<T, 128, 1, false>(p, grid, a, s);
    else
        launch_rows<T, 256, 1, false>(p, grid, a, s);
}

// Wavefronts per item: as many as fit the chip's registers at once, no more than the item has tiles.  Two per
// SIMD up to 128 channels, one with more (256 registers and up to 208 accumulation registers each): shared out
// for two, a second round of workgroups started behind the first (256 channels, 32/8 heads, 3 prompts of
// 700 tokens x 40 samples: fp32 91 -> 74 us, bf16 53 -> 40; of 58 shapes three fp32 ones lost 9 %).
// Suffix items find half of the prefix items' places taken (fp32, 16 samples of a 2k prompt, suffixes of up to 256:
// four wavefronts a 64-token chunk 23.3 us, two 21.5; 20 samples x 8 heads x 100 tokens keep four, 25.5 / 26.4;
// 32 samples x 8 heads with 64 channels lose a little, 23.9 / 24.2).
int share_of(long long items, int tiles, int head_dim, long long prefix_waves = 0)
{
    const long long places = head_dim > 128 ? 1024 : 2048 - prefix_waves / 2;
    int share = 1;
    while (2 * share <= kWaves && 2 * share <= tiles && items * share * 2 <= places)
        share *= 2;
    return share;
}

}  // namespace

hipError_t launch_attn_rows(const AttnParams& p, bool prefix, bool suffix, hipStream_t s)
{
    prefix = prefix && p.num_prefix_splits > 0;
    suffix = suffix && p.num_suffix_chunks > 0;
    if (!prefix && !suffix)
        return hipSuccess;
    const long long max_rows = (long long)p.max_spp * p.G;
    const int block = plan::rows_per_block(p.D, max_rows);
    const int tile = p.dtype == 0 ? 16 : 32;
    const long long rowblocks = (max_rows + block - 1) / block;
    const long long units = prefix ? (long long)p.num_prefix_splits * p.B * p.Hkv : 0;
    const long long suffix_items = suffix ? (long long)((p.G + 15) / 16) * p.Hkv * p.num_suffix_chunks * p.N : 0;
    RowsLaunch a;
    a.prefix_share = share_of(rowblocks * units, p.prefix_split_tokens / tile, p.D);
    const long long prefix_waves = rowblocks * units * a.prefix_share;
    a.suffix_share = share_of(suffix_items, p.suffix_chunk_tokens / tile, p.D, prefix_waves < 2048 ? prefix_waves : 2048);
    const int per_p = kWaves / a.prefix_share, per_s = kWaves / a.suffix_share;
    const long long prefix_blocks = units * ((rowblocks + per_p - 1) / per_p);
    const long long blocks = prefix_blocks + (suffix_items + per_s - 1) / per_s;
    if (blocks > 0x7fffffffLL || suffix_items > 0x7fffffffLL)
        return hipErrorInvalidValue;
    a.suffix_items = (unsigned)suffix_items;
    a.g_inv = p.G > 1 ? (unsigned)((1ll << 32) / p.G) : 0xffffffffu;
    a.prefix_rowblocks = (int)rowblocks;
    a.prefix_blocks = (int)prefix_blocks;
    const bool ring = suffix && plan::rows_through_lds(p.dtype, p.D, p.suffix_chunk_tokens, a.suffix_share);
    if (p.dtype == 0)
        launch_rows_dim<float>(p, block / 16, false, (unsigned)blocks, a, s);
    else
        launch_rows_dim<uint16_t>(p, block / 16, ring, (unsigned)blocks, a, s);
    return hipGetLastError();
}

}  // namespace spd
