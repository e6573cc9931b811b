// Log-sum-exp merge of partial softmax states (prefix splits and suffix chunks) into
// the normalised attention output.  With states (m_i, l_i, out_i = acc_i / l_i):
//   m = max m_i,  w_i = l_i 2^(m_i - m),  l = sum w_i,  out = sum w_i out_i / l,
//   lse = (m + log2 l) ln 2.
// This is the rescaling step of the paper's online-softmax recurrence (App., attn
// task 2: `ExpMaxDiff`, `WeightedSumSingle`, `WeightedSumDouble`, `Div`) applied to
// blocks instead of single tokens.  Empty ranges carry l = 0 and weight 0, so the initial state
// (-inf, 0, 0) is the identity.
#include "spd_internal.h"

#include <hip/hip_fp16.h>

namespace spd {
namespace {

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u)
        return (uint16_t)((u >> 16) | 0x40);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

constexpr int kMergeWaves = 4;   // wavefronts per workgroup

// 16 bytes of a partial output: 8 channels of fp16 or 4 of fp32.
template <bool HALF> struct PartVec {
    static constexpr int kChannels = HALF ? 8 : 4;
    static __device__ __forceinline__ void widen(const uint4& v, float (&f)[kChannels])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (HALF) {
                const float2 a = __half22float2(*reinterpret_cast<const __half2*>(&w[i]));
                f[2 * i] = a.x;
                f[2 * i + 1] = a.y;
            } else {
                f[i] = __uint_as_float(w[i]);
            }
        }
    }
};

// CL lanes own the 16-byte pieces of a row (a power of two that covers them); GROUPS such groups of
// lanes share the row's slots (group g takes slots g, g + GROUPS, ...) and add their sums with shuffles; a
// wavefront takes 64 / (CL GROUPS) rows.  The lanes of a row also take its (m, l) pairs, and hand
// their weights round with shuffles, so there is no LDS and no barrier.  BATCH is the number of parts a
// lane requests at a time.
//   few rows: all 64 lanes on one row (up to 128 slots, two pairs per lane).  Bound: latency, i.e. one round
//     trip for everything (the pairs and the first BATCH parts of every lane are requested together,
//     from clamped places rather than under branches) and the launch.
//   many rows of at most eight slots: one group per row.  Bound: HBM (partial states) from some 16384 rows
//     on, latency below.
// Measured in replayed graphs (before: 32 threads per row, up to 32 guarded loads each, weights through
// LDS): 512 rows x 20 slots 6.1 -> 3.6 us, 2048 x 22 6.6 -> 4.7, 13312 x 26 18.0 -> 10.1,
// 16 x 5 (fp32) 3.7 -> 2.5; 32768 x 8 14.4 -> 14.2 (16.2 with all 64 lanes on one row).
template <bool HALF, int CL, int GROUPS, int BATCH>
__global__ __launch_bounds__(kMergeWaves * 64) void attn_merge_kernel(AttnParams p)
{
    constexpr int kLanes = CL * GROUPS, kRows = 64 / kLanes, kCh = PartVec<HALF>::kChannels;
    constexpr int kPairs = kLanes == 64 ? 2 : 1;   // (m, l) pairs per lane
    const int lane = threadIdx.x & 63, mine = lane % kLanes, c = lane % CL, g = mine / CL;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = ((int)blockIdx.x * kMergeWaves + wave) * kRows + lane / kLanes;
    const bool row_ok = row < p.N * p.Hq;
    // Every slot of the row holds an (m, l) pair: the pass that owns a slot stores l = 0 when its
    // token range is empty (a prefix split past the group's length, a suffix chunk past the
    // sample's), and leaves the slot's output part unwritten.  The row therefore needs no lengths
    // here; a slot with l = 0 gets weight 0 and its output part, though loaded, is not used.
    const int S = p.num_slots;
    const long long base = part_index(p, row_ok ? row : 0, 0);
    const bool ch_ok = kCh * c < p.D;
    const char* parts = (const char*)p.part_acc + (base * p.D + (ch_ok ? kCh * c : 0)) * (HALF ? 2 : 4);
    const unsigned part_bytes = (unsigned)p.D * (HALF ? 2u : 4u);
    uint4 v[BATCH];
    auto request = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            v[u] = *reinterpret_cast<const uint4*>(parts + (size_t)((unsigned)min(s0 + u * GROUPS + g, S - 1) * part_bytes));
    };
    float2 ml[kPairs];
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < kPairs; ++k) {
        ml[k] = make_float2(-INFINITY, 0.f);
        if (mine + kLanes * k < S)
            ml[k] = p.part_ml[base + mine + kLanes * k];
    }
    if (S > 0)
        request(0);
#pragma unroll
    for (int k = 0; k < kPairs; ++k)
        m = ml[k].y > 0.f ? fmaxf(m, ml[k].x) : m;
#pragma unroll
    for (int o = kLanes >> 1; o > 0; o >>= 1)
        m = fmaxf(m, __shfl_xor(m, o));
    float w[kPairs], l = 0.f;
#pragma unroll
    for (int k = 0; k < kPairs; ++k) {
        w[k] = ml[k].y > 0.f ? ml[k].y * __builtin_amdgcn_exp2f(ml[k].x - m) : 0.f;
        l += w[k];
    }
#pragma unroll
    for (int o = kLanes >> 1; o > 0; o >>= 1)
        l += __shfl_xor(l, o);
    float acc[kCh];
#pragma unroll
    for (int e = 0; e < kCh; ++e)
        acc[e] = 0.f;
    for (int s0 = 0; s0 < S; s0 += BATCH * GROUPS) {
        if (s0 > 0)
            request(s0);
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = s0 + u * GROUPS + g;
            float ws = __shfl(w[0], (lane & ~(kLanes - 1)) + (s & (kLanes - 1)));
            if (kPairs == 2 && S > kLanes)
                ws = s < kLanes ? ws : __shfl(w[1], s & (kLanes - 1));
            float f[kCh];
            PartVec<HALF>::widen(v[u], f);
            if (ws != 0.f && s < S) {
#pragma unroll
                for (int e = 0; e < kCh; ++e)
                    acc[e] = fmaf(f[e], ws, acc[e]);
            }
        }
    }
#pragma unroll
    for (int o = CL; o < kLanes; o <<= 1)
#pragma unroll
        for (int e = 0; e < kCh; ++e)
            acc[e] += __shfl_xor(acc[e], o);
    const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
    for (int e = 0; e < kCh; ++e)
        acc[e] *= inv;
    if (g == 0 && ch_ok && row_ok) {
        const long long at = (long long)row * p.D + kCh * c;
        if constexpr (HALF) {
            uint4 o;
            o.x = (uint32_t)f32_to_bf16_rne(acc[0]) | ((uint32_t)f32_to_bf16_rne(acc[1]) << 16);
            o.y = (uint32_t)f32_to_bf16_rne(acc[2]) | ((uint32_t)f32_to_bf16_rne(acc[3]) << 16);
            o.z = (uint32_t)f32_to_bf16_rne(acc[4]) | ((uint32_t)f32_to_bf16_rne(acc[5]) << 16);
            o.w = (uint32_t)f32_to_bf16_rne(acc[6]) | ((uint32_t)f32_to_bf16_rne(acc[7]) << 16);
            *reinterpret_cast<uint4*>((uint16_t*)p.out + at) = o;
        } else {
            *reinterpret_cast<float4*>((float*)p.out + at) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
    }
    if (p.lse && mine == 0 && row_ok)
        p.lse[row] = l > 0.f ? (m + __log2f(l)) * kLn2 : -INFINITY;
}

template <bool HALF, int CL, int GROUPS, int BATCH>
void launch_merge_kernel(const AttnParams& p, hipStream_t s)
{
    constexpr int kRowsPerBlock = kMergeWaves * 64 / (CL * GROUPS);
    const dim3 grid((unsigned)(((long long)p.N * p.Hq + kRowsPerBlock - 1) / kRowsPerBlock));
    hipLaunchKernelGGL((attn_merge_kernel<HALF, CL, GROUPS, BATCH>), grid, dim3(kMergeWaves * 64), 0, s, p);
}

template <bool HALF, int CL>
void launch_merge_cl(const AttnParams& p, hipStream_t s)
{
    // With up to eight slots a lane requests a row's whole column at once, so sharing the slots out only adds
    // wavefronts, which pays while there are few rows.  Shared / not shared, bf16, 128 channels: 1024 rows
    // x 2 slots 3.8 / 3.6 us, x 5 3.8 / 3.9, 2048 x 5 4.0 / 4.0, 4096 x 2 4.6 / 3.7, x 8 4.6 / 4.1,
    // 6144 x 5 5.3 / 4.3, 16384 x 8 9.1 / 7.0, 32768 x 8 16.2 / 14.2 (fp32 and other widths cross there too).
    if (CL < 64 && p.num_slots <= 8 && (long long)p.N * p.Hq >= (p.num_slots <= 4 ? 1024 : 2048)) {
        if (p.num_slots <= 4)
            launch_merge_kernel<HALF, CL, 1, 4>(p, s);
        else
            launch_merge_kernel<HALF, CL, 1, 8>(p, s);
        return;
    }
    const int per_lane = (p.num_slots + 64 / CL - 1) / (64 / CL);
    if (per_lane <= 2)
        launch_merge_kernel<HALF, CL, 64 / CL, 2>(p, s);
    else if (per_lane <= 4)
        launch_merge_kernel<HALF, CL, 64 / CL, 4>(p, s);
    else
        launch_merge_kernel<HALF, CL, 64 / CL, 8>(p, s);
}

}  // namespace

// Partial outputs are fp16 exactly when the result is bf16 (p.part_half).
hipError_t launch_attn_merge(const AttnParams& p, hipStream_t s)
{
    const int pieces = p.D * (p.part_half ? 2 : 4) / 16;
    if (p.part_half) {
        if (pieces <= 8) launch_merge_cl<true, 8>(p, s);
        else if (pieces <= 16) launch_merge_cl<true, 16>(p, s);
        else launch_merge_cl<true, 32>(p, s);
    } else {
        if (pieces <= 8) launch_merge_cl<false, 8>(p, s);
        else if (pieces <= 16) launch_merge_cl<false, 16>(p, s);
        else if (pieces <= 32) launch_merge_cl<false, 32>(p, s);
        else launch_merge_cl<false, 64>(p, s);
    }
    return hipGetLastError();
}

}  // namespace spd
