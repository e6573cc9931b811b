// Temperature / nucleus / inverse-CDF token sampler.
//
// Two paths.  The sliced path (below: two stream-ordered kernels) reads a row from HBM once, leaves
// what the row-level step needs in the workspace, and finds the exact nucleus threshold without
// sorting.  The whole-row routine (one workgroup per row, every pass from memory) covers what the
// sliced path does not take: vocabularies of fewer than 4 logits, rows with more than 512 logits at a threshold that are
// nearly but not quite equal, rows with a cut at an infinite temperature, and, among rows that do not start on a
// 16-byte boundary, short ones.
//
// Probabilities are p_i = 2^((x_i - max) c) with c = log2(e)/T carried as hi + lo floats, by one routine (prob)
// but for two things: the scan's mass of a slice splits c in another place (so that its second part is positive) and is
// relative to the slice's maximum, and the bins of the row-level step use c_hi alone.  Bins only point at a place:
// what lies above it and in it is then summed logit by logit in fp64, and a threshold that those sums do not bear out
// sends the row to the whole-row routine.  Masses of slices and of the segments that the walk goes through are fp64 sums of
// groups of four in fp32.  The whole-row routine keeps what is not below the threshold by the bit pattern of p, the sliced
// path by the logit, so that all ties with the threshold are kept.  A list's order depends on which wavefront reserved its
// places first; with it the last bits of fp64 sums can differ from call to call, and nothing else.
#include "spd_internal.h"

#include <type_traits>

namespace spd {
namespace {

constexpr int kBlock = 512;
constexpr int kWaves = kBlock / 64;
constexpr int kBins = 2048;
constexpr int kSeg = 256;           // elements per wave per tile (64 lanes x 4)
constexpr int kTile = kWaves * kSeg;  // elements per block iteration (64 lanes x 4 per wave)
constexpr int kMaxSegments = 1024;    // vocab <= 262144

struct RowScale {
    float max_x, c_hi, c_lo;
};

__device__ __forceinline__ float prob(float x, const RowScale& r)
{
    const float d = x - r.max_x;
    const float y = __builtin_fmaf(d, r.c_hi, d * r.c_lo);
    // (a logit of -inf: where c_lo is negative, as at temperatures 0.4 and 0.7, the two terms are infinities of
    // opposite sign; the maximum takes the zero)
    return fmaxf(__builtin_amdgcn_exp2f(y), 0.f);
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    for (int o = 32; o > 0; o >>= 1)
        v += __shfl_xor(v, o);
    return v;
}

// ---- scans and reductions across a wavefront without LDS traffic (data-parallel primitives: shifts inside
// rows of 16 lanes, then the last lane of a row broadcast into the rows after it).  All 64 lanes
// must be active.  A lane that receives nothing keeps `none`.
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned dpp_u32(unsigned none, unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_f64(double v)  // 0.0 where nothing arrives
{
    const unsigned lo = dpp_u32<CTRL, ROWS>(0u, (unsigned)__double2loint(v)), hi = dpp_u32<CTRL, ROWS>(0u, (unsigned)__double2hiint(v));
    return __hiloint2double((int)hi, (int)lo);
}
constexpr int kShr1 = 0x111, kShr2 = 0x112, kShr4 = 0x114, kShr8 = 0x118, kBcast15 = 0x142, kBcast31 = 0x143;

// A value that is the same in every lane, moved to a scalar register.
__device__ __forceinline__ float uniform(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// The same value in a scalar register, for the compiler another one: what is formed from it is formed here, not ahead of the loop
// around, where it would take vector registers (of uniform values too: scalar arithmetic has no floats).
__device__ __forceinline__ float here(float v)
{
    int s = __builtin_amdgcn_readfirstlane(__float_as_int(v));
    asm volatile("" : "+s"(s));
    return __int_as_float(s);
}
__device__ __forceinline__ double here(double v)
{
    int lo = __builtin_amdgcn_readfirstlane(__double2loint(v)), hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
    asm volatile("" : "+s"(lo), "+s"(hi));
    return __hiloint2double(hi, lo);
}

// Inclusive scan over the lanes.
__device__ __forceinline__ double wave_scan_f64(double v)
{
    v += dpp_f64<kShr1, 0xf>(v);
    v += dpp_f64<kShr2, 0xf>(v);
    v += dpp_f64<kShr4, 0xf>(v);
    v += dpp_f64<kShr8, 0xf>(v);
    v += dpp_f64<kBcast15, 0xa>(v);
    v += dpp_f64<kBcast31, 0xc>(v);
    return v;
}
__device__ __forceinline__ unsigned wave_scan_u32(unsigned v)
{
    v += dpp_u32<kShr1, 0xf>(0u, v);
    v += dpp_u32<kShr2, 0xf>(0u, v);
    v += dpp_u32<kShr4, 0xf>(0u, v);
    v += dpp_u32<kShr8, 0xf>(0u, v);
    v += dpp_u32<kBcast15, 0xa>(0u, v);
    v += dpp_u32<kBcast31, 0xc>(0u, v);
    return v;
}
__device__ __forceinline__ float wave_scan_f32(float v)
{
    auto add = [](float a, unsigned b) { return a + __uint_as_float(b); };
    v = add(v, dpp_u32<kShr1, 0xf>(0u, __float_as_uint(v)));
    v = add(v, dpp_u32<kShr2, 0xf>(0u, __float_as_uint(v)));
    v = add(v, dpp_u32<kShr4, 0xf>(0u, __float_as_uint(v)));
    v = add(v, dpp_u32<kShr8, 0xf>(0u, __float_as_uint(v)));
    v = add(v, dpp_u32<kBcast15, 0xa>(0u, __float_as_uint(v)));
    v = add(v, dpp_u32<kBcast31, 0xc>(0u, __float_as_uint(v)));
    return v;
}
// Reductions: the same value in every lane.
template <typename F> __device__ __forceinline__ unsigned wave_reduce_u32(unsigned v, unsigned none, F f)
{
    v = f(v, dpp_u32<kShr1, 0xf>(none, v));
    v = f(v, dpp_u32<kShr2, 0xf>(none, v));
    v = f(v, dpp_u32<kShr4, 0xf>(none, v));
    v = f(v, dpp_u32<kShr8, 0xf>(none, v));
    v = f(v, dpp_u32<kBcast15, 0xa>(none, v));
    v = f(v, dpp_u32<kBcast31, 0xc>(none, v));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ float wave_max_f32(float v)
{
    return __uint_as_float(wave_reduce_u32(__float_as_uint(v), 0xff800000u /* -inf */, [](unsigned a, unsigned b) {
        return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
    }));
}
__device__ __forceinline__ unsigned wave_min_u32(unsigned v)
{
    return wave_reduce_u32(v, 0xffffffffu, [](unsigned a, unsigned b) { return min(a, b); });
}
__device__ __forceinline__ unsigned wave_max_u32(unsigned v)
{
    return wave_reduce_u32(v, 0u, [](unsigned a, unsigned b) { return max(a, b); });
}

// Block-wide sum in fp64 with a fixed reduction tree (deterministic).
__device__ double block_sum_f64(double v, double* scratch /* kWaves */)
{
    v = wave_sum_f64(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        scratch[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w)
        t += scratch[w];
    return t;
}

// Chooses the refinement bin: the highest non-empty bin b whose cumulative mass
// c(b) = above + sum_{b' >= b} hist[b'] reaches `need`.  If rounding leaves even the
// total short of `need`, the lowest non-empty bin is taken (everything is kept).
// Results are left in *bin_out and *above_out (mass strictly above the chosen bin).
// Thread t owns the kBinsPerThread consecutive bins just below kBins - t * kBinsPerThread.
constexpr int kBinsPerThread = kBins / kBlock;

__device__ void pick_bin(const double* hist, double above, double need, int* bin_out,
                         int* low_out, double* above_out, double* scratch /* kWaves */)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int top = kBins - 1 - kBinsPerThread * tid;
    __syncthreads();  // callers may have just used `scratch` and the output slots
    double h[kBinsPerThread];
    double own = 0.0;
#pragma unroll
    for (int k = 0; k < kBinsPerThread; ++k) {
        h[k] = hist[top - k];
        own += h[k];
    }
    double incl = own;
    for (int o = 1; o < 64; o <<= 1) {
        const double up = __shfl_up(incl, o);
        if (lane >= o)
            incl += up;
    }
    if (tid == 0) {
        *bin_out = -1;
        *low_out = kBins;
    }
    if (lane == 63)
        scratch[wave] = incl;
    __syncthreads();
    double before = above + (incl - own);
#pragma unroll 1  // (unrolled it takes registers that the row-level kernels do not have)
    for (int w = 0; w < wave; ++w)
        before += scratch[w];
    int best = -1, low = kBins;
#pragma unroll
    for (int k = 0; k < kBinsPerThread; ++k) {
        if (h[k] > 0.0) {
            low = top - k;
            if (best < 0 && before + h[k] >= need)
                best = top - k;
        }
        if (best < 0)
            before += h[k];
    }
    // `before` now holds the mass strictly above `best` (when this thread found one)
    if (best >= 0)
        atomicMax(bin_out, best);
    if (low < kBins)
        atomicMin(low_out, low);
    __syncthreads();
    const int chosen = *bin_out >= 0 ? *bin_out : (*low_out < kBins ? *low_out : 0);
    const bool fallback = *bin_out < 0;
    __syncthreads();
    if (!fallback) {
        if (best == chosen)
            *above_out = before;
    } else if (chosen <= top && chosen > top - kBinsPerThread) {
        // everything above the lowest non-empty bin
        double b2 = above + (incl - own);
#pragma unroll 1
        for (int w = 0; w < wave; ++w)
            b2 += scratch[w];
        for (int k = 0; k < top - chosen; ++k)
            b2 += h[k];
        *above_out = b2;
    }
    if (tid == 0)
        *bin_out = chosen;
    __syncthreads();
}

// Shared-memory arrays of the row routines (one instance per workgroup).
struct RowLds {
    double hist[kBins];
    double scratch[2 * kWaves];  // block sums and scans
    double seg_mass[kMaxSegments];
    float red_f[kWaves];
    int red_i[kWaves];
    int sh_low;
    int sh_bin;
    double sh_above;
    int sh_token;
};

// Whole-row routine for one workgroup of kBlock threads: every pass reads the row from
// global memory.  Used when the sliced kernel cannot take a row (very large vocabularies,
// candidate overflow).
__device__ __forceinline__ void sample_row_from_memory(const SamplerParams& sp, long long r, RowLds& L)
{
    double* hist = L.hist;
    double* scratch = L.scratch;
    double* seg_mass = L.seg_mass;
    float* red_f = L.red_f;
    int* red_i = L.red_i;
    int& sh_low = L.sh_low;
    int& sh_bin = L.sh_bin;
    double& sh_above = L.sh_above;
    int& sh_token = L.sh_token;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* __restrict__ x = sp.logits + r * sp.stride;
    const int V = (int)sp.vocab;
    const float T = sp.temperature[r];

    // ---- pass 1: maximum and its lowest index -------------------------------------------
    float mx = -INFINITY;
    int mi = 0x7fffffff;
    for (int i = tid; i < V; i += kBlock) {
        const float v = x[i];
        if (v > mx) {
            mx = v;
            mi = i;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(mx, o);
        const int oi = __shfl_xor(mi, o);
        if (ov > mx || (ov == mx && oi < mi)) {
            mx = ov;
            mi = oi;
        }
    }
    if (lane == 0) {
        red_f[wave] = mx;
        red_i[wave] = mi;
    }
    __syncthreads();
    mx = red_f[0];
    mi = red_i[0];
    for (int w = 1; w < kWaves; ++w) {
        if (red_f[w] > mx || (red_f[w] == mx && red_i[w] < mi)) {
            mx = red_f[w];
            mi = red_i[w];
        }
    }
    if (T == 0.f) {
        if (tid == 0)
            sp.tokens[r] = mi;
        return;
    }

    RowScale rs;
    rs.max_x = mx;
    {
        const double c = 1.4426950408889634 / (double)T;
        rs.c_hi = (float)c;
        rs.c_lo = (float)(c - (double)rs.c_hi);
    }

    // ---- filters ahead of the nucleus: a lower bound `lb_bits` on the bit pattern of p ----------
    // (p > 0, so patterns order like values.)  min-p: p >= min_p, and the maximum has p = 1.
    // top-k: the k-th largest pattern among what min-p left, found by radix select on counts;
    // every tie with it is kept.
    const float top_p = sp.top_p[r];
    const bool cut = top_p < 1.f;
    const float min_p = sp.min_p ? sp.min_p[r] : 0.f;
    const int top_k = sp.top_k ? sp.top_k[r] : 0;
    uint32_t lb_bits = min_p > 0.f ? __float_as_uint(min_p) : 0u;

    // Radix select over the patterns >= lb (bits 30..20, 19..9, 8..0): the highest pattern whose
    // upper set reaches `need`, counting tokens (`by_count`) or summing their probabilities.
    auto select = [&](bool by_count, double need, uint32_t lb) -> uint32_t {
        uint32_t prefix = 0u;
        double above = 0.0;
        for (int level = 0; level < 3; ++level) {
            const int shift = level == 0 ? 20 : level == 1 ? 9 : 0;
            const int bits = level == 2 ? 9 : 11;
            for (int b = tid; b < kBins; b += kBlock)
                hist[b] = 0.0;
            __syncthreads();
            for (int i = tid; i < V; i += kBlock) {
                const float pv = prob(x[i], rs);
                const uint32_t u = __float_as_uint(pv) & 0x7fffffffu;
                if (u >= lb && (level == 0 || (u >> (shift + bits)) == prefix))
                    atomicAdd(&hist[(u >> shift) & ((1u << bits) - 1u)], by_count ? 1.0 : (double)pv);
            }
            __syncthreads();
            pick_bin(hist, above, need, &sh_bin, &sh_low, &sh_above, scratch);
            prefix = (prefix << bits) | (uint32_t)sh_bin;
            above = sh_above;
            __syncthreads();
        }
        return prefix;
    };
    if (top_k > 0)
        lb_bits = max(lb_bits, select(true, (double)top_k, lb_bits));

    // ---- pass 2: mass of what the filters left; nucleus threshold among it --------------------------
    double part = 0.0;
    {
        float acc = 0.f;
        int cnt = 0;
        for (int i = tid; i < V; i += kBlock) {
            const float pv = prob(x[i], rs);
            if ((__float_as_uint(pv) & 0x7fffffffu) < lb_bits)
                continue;
            acc += pv;
            if (++cnt == 32) {  // bound the fp32 run length before widening
                part += (double)acc;
                acc = 0.f;
                cnt = 0;
            }
        }
        part += (double)acc;
    }
    const double S = block_sum_f64(part, scratch);

    uint32_t tau_bits = lb_bits;  // keep everything the filters left
    double Z = S;
    if (cut)
        tau_bits = max(lb_bits, select(false, (double)top_p * S, lb_bits));

    // ---- pass 3: kept mass per 256-element segment, in vocabulary order -----------------
    const int num_tiles = (V + kTile - 1) / kTile;
    double z_part = 0.0;
    for (int tile = 0; tile < num_tiles; ++tile) {
        const int base = tile * kTile + wave * kSeg + lane * 4;
        float s4 = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = base + k;
            if (i < V) {
                const float pv = prob(x[i], rs);
                if (__float_as_uint(pv) >= tau_bits)
                    s4 += pv;
            }
        }
        const double ws = wave_sum_f64((double)s4);
        if (lane == 0)
            seg_mass[tile * kWaves + wave] = ws;  // vocab <= kMaxSegments * kSeg checked on the host
        z_part += (lane == 0) ? ws : 0.0;
    }
    Z = block_sum_f64(z_part, scratch);
    const double target = (double)sp.uniforms[r] * Z;

    // ---- scan the segments (one wave), then walk inside the hit segment ------------------
    if (wave == 0) {
        const int nseg = num_tiles * kWaves;
        const int per = (nseg + 63) / 64;  // consecutive segments per lane
        double mine = 0.0;
        for (int k = 0; k < per; ++k) {
            const int sidx = lane * per + k;
            if (sidx < nseg)
                mine += seg_mass[sidx];
        }
        double incl = mine;
        for (int o = 1; o < 64; o <<= 1) {
            const double up = __shfl_up(incl, o);
            if (lane >= o)
                incl += up;
        }
        const double before_lane = incl - mine;
        // first lane whose inclusive mass exceeds the target
        const unsigned long long hit = __ballot(incl > target);
        int seg = -1;
        double before = 0.0;
        if (hit) {
            const int hl = __ffsll((long long)hit) - 1;
            double run = __shfl(before_lane, hl);
            // walk that lane's few segments (every lane does it redundantly)
            for (int k = 0; k < per; ++k) {
                const int sidx = hl * per + k;
                if (sidx >= nseg)
                    break;
                const double sm = seg_mass[sidx];
                if (run + sm > target) {
                    seg = sidx;
                    before = run;
                    break;
                }
                run += sm;
            }
        }
        int token = -1;
        if (seg >= 0) {
            const int base = seg * kSeg + lane * 4;
            float pv[4];
            bool keep[4];
            float s4 = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = base + k;
                pv[k] = 0.f;
                keep[k] = false;
                if (i < V) {
                    const float q = prob(x[i], rs);
                    if (__float_as_uint(q) >= tau_bits) {
                        pv[k] = q;
                        keep[k] = true;
                        s4 += q;
                    }
                }
            }
            double incl2 = (double)s4;
            for (int o = 1; o < 64; o <<= 1) {
                const double up = __shfl_up(incl2, o);
                if (lane >= o)
                    incl2 += up;
            }
            double run = before + incl2 - (double)s4;
            int cand = 0x7fffffff;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (keep[k]) {
                    run += (double)pv[k];
                    if (run > target && cand == 0x7fffffff)
                        cand = base + k;
                }
            }
            for (int o = 32; o > 0; o >>= 1)
                cand = min(cand, __shfl_xor(cand, o));
            if (cand != 0x7fffffff)
                token = cand;
        }
        if (lane == 0)
            sh_token = token;
    }
    __syncthreads();
    if (sh_token >= 0) {
        if (tid == 0)
            sp.tokens[r] = sh_token;
        return;
    }
    // Rounding let the walk finish without crossing: return the last kept index.
    int last = -1;
    for (int i = tid; i < V; i += kBlock)
        if (__float_as_uint(prob(x[i], rs)) >= tau_bits)
            last = max(last, i);
    for (int o = 32; o > 0; o >>= 1)
        last = max(last, __shfl_xor(last, o));
    __syncthreads();
    if (lane == 0)
        red_i[wave] = last;
    __syncthreads();
    if (tid == 0) {
        int best = -1;
        for (int w = 0; w < kWaves; ++w)
            best = max(best, red_i[w]);
        sp.tokens[r] = best;
    }
}

// =============================================================================================
// Sliced path: a row is cut into `slices` contiguous pieces of at most kSliceMax elements and
// handled by two kernels in stream order; no workgroup ever waits for another and there are no
// cross-workgroup counters.
//
//   scan    (rows x slices)  the one pass over the logits.  A workgroup holds its slice in
//           registers and leaves behind what the row-level step can need from it: the slice
//           maximum (and its lowest index), the slice's mass relative to that maximum, and the
//           list of the logits in a window [x_lo, x_hi) that the nucleus cut probably falls
//           into, with the mass above the window.  Where the window lies is a guess from every
//           fourth element: counts over bins of a quarter octave name the place where the mass
//           below is 1 - top_p of the slice's own (whose sum is exact).  The list begins at the top
//           (x_hi = +inf) where what lies above the cut fits it.
//   finish  (rows)  knows the row's mass S.  It bins the listed logits over the few octaves that the cut
//           must lie in, picks the bin that takes the running mass across top_p S, checks that every
//           slice's window reaches around that bin (a slice whose window does not is read a second
//           time, all of it), sums up exactly what lies above the bin, and tells the few logits inside
//           it apart directly.  Then the slice that holds u Z follows from the slices' kept masses; it is
//           read again, and the walk goes on in registers: its 256-element segments, then the elements
//           of one.
//           Rows with a min-p or top-k filter (a second instantiation of the kernel, launched in place
//           of the first when filter arrays are given, takes both kinds of row): the scan kernel lists
//           such a row from the top as far as its filters are likely to reach; the k-th largest is
//           found as the cut is, by counts instead of masses.
//
// With the row statistics exchanged through memory between two kernels, plain stores and loads do.
// =============================================================================================
constexpr int kIter = kBlock * 4;         // elements one float4 per thread covers
constexpr int kSliceMax = 8 * kIter;      // elements per workgroup: 8 float4 per thread
constexpr int kMaxSlices = 16;
constexpr int kSegPerSlice = kSliceMax / kSeg;  // 64
constexpr int kListCap = 5248;            // logits that a slice may list (21 KB of workspace with its statistics)
static_assert(kMaxSlices * kSegPerSlice <= kMaxSegments, "segment table too small");

struct SliceStat {
    float max_x;
    int argmax;
    double mass;       // of the whole slice, relative to max_x
    double above;      // of what lies at or above x_hi, relative to max_x
    float x_lo, x_hi;  // listed: x_lo <= x < x_hi (x_lo = -FLT_MAX: whatever lies below x_hi)
    int count;         // listed logits; -1: more than the list holds
    float x_cut;       // about where the slice's own cut lies
};
static_assert(sizeof(SliceStat) <= 64, "slice statistics are kept 64 bytes apart");

__host__ __device__ inline size_t sliced_row_bytes(int slices)
{
    return (size_t)slices * (64 + (size_t)kListCap * 4);
}

struct RowWs {
    char* stat;   // [slices] SliceStat, 64 B apart
    float* list;  // [slices][kListCap]
};

__device__ __forceinline__ RowWs row_ws(char* base, long long row, int slices)
{
    RowWs w;
    w.stat = base + row * sliced_row_bytes(slices);
    w.list = (float*)(w.stat + (size_t)slices * 64);
    return w;
}

__device__ __forceinline__ SliceStat* stat_at(const RowWs& w, int s) { return (SliceStat*)(w.stat + (size_t)s * 64); }

// Monotone map of a float onto unsigned integers (larger float -> larger key), and back.
__device__ __forceinline__ uint32_t order_key(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k); }

struct RowConst {
    float c_hi, c_lo;
    double cd;
};

__device__ __forceinline__ RowConst row_const(float T)
{
    RowConst k;
    k.cd = 1.4426950408889634 / (double)T;
    k.c_hi = (float)k.cd;
    k.c_lo = (float)(k.cd - (double)k.c_hi);
    return k;
}

// Slice [e0, e1) of a row.
struct SliceRange {
    int e0, e1;
};

__device__ __forceinline__ SliceRange slice_range(int slice, int slice_elems, int V)
{
    SliceRange g;
    g.e0 = slice * slice_elems;
    g.e1 = min(V, g.e0 + slice_elems);
    return g;
}

// Four logits at once; rows of a vocabulary that is not a multiple of 4 need not begin on a 16-byte boundary (the
// load asks for 4 bytes only).  STREAM: not kept in the caches (the pass of launch_sampler over logits that do not fit them).
template <bool STREAM> __device__ __forceinline__ float4 load4(const float* at)
{
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const f32x4 v = STREAM ? __builtin_nontemporal_load((const f32x4*)at) : *(const f32x4*)at;
    return make_float4(v[0], v[1], v[2], v[3]);
}

// Loads a slice into 32 registers per thread, element e0 + j kIter + 4 tid + k in register 4 j + k.  Every load is
// unconditional (what would reach past the slice reads its last four logits), so that the hardware's in-order load
// counter stays exact for the compiler and later loads need not wait for these.
// mask_four, applied where the values are first needed, moves the logits of a float4 that the slice's end cuts
// to their places and puts -inf behind them.  Every slice holds four logits at least (the host sends
// shorter rows to the whole-row kernel, and slices are never shorter than about 2000).
#define SPD_LOAD_SLICE(STREAM, xv, xr, g, tid)                                          \
    _Pragma("unroll") for (int j = 0; j < 8; ++j)                                       \
    {                                                                                   \
        const float4 v_ = load4<STREAM>((xr) + min((g).e0 + j * kIter + (tid) * 4, (g).e1 - 4)); \
        (xv)[4 * j] = v_.x;                                                             \
        (xv)[4 * j + 1] = v_.y;                                                         \
        (xv)[4 * j + 2] = v_.z;                                                         \
        (xv)[4 * j + 3] = v_.w;                                                         \
    }
// a .. d were read `over` places too early: moves them there, -inf behind the last.
__device__ __forceinline__ void mask_four(float& a, float& b, float& c, float& d, int over)
{
    const bool one = over > 0 && (over & 1), two = over > 0 && (over & 2), out = over >= 4;
    a = one ? b : a;
    b = one ? c : b;
    c = one ? d : c;
    d = one ? -INFINITY : d;
    a = two ? c : a;
    b = two ? d : b;
    c = two ? -INFINITY : c;
    d = two ? -INFINITY : d;
    a = out ? -INFINITY : a;
    b = out ? -INFINITY : b;
    c = out ? -INFINITY : c;
    d = out ? -INFINITY : d;
}

// Barrier between phases that exchange data through LDS only: waits for this wavefront's LDS
// traffic, not for its global loads and stores (a __syncthreads would drain those too, and the
// slice's logits and the published results are still in flight at most barriers of these kernels).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---- kernel 1: the pass over the logits --------------------------------------------------------------
constexpr int kGuessBins = 256;    // a quarter octave of p each, counted down from the slice's maximum
constexpr int kStrip = 16;         // logits a lane may list per half of its slice: all of them

struct ScanLds {
    unsigned hist[kGuessBins];     // every fourth element, by bin below the maximum
    float cum[kGuessBins + 1], below[kGuessBins + 1];  // [b]: count and mass of the first b bins from the top
    float strip[kStrip][kBlock];   // each lane's listed logits
    double mass[kWaves];
    float red_f[kWaves];
    float squares[kWaves];         // (not red_f again: a wavefront may still be reading the maxima there)
    int red_i[kWaves];
    float x_lo, x_hi;
    unsigned emitted;              // places reserved in the slice's list so far
};

constexpr float kListLeast = 500.f;               // a slice lists at least about that many of its largest logits
constexpr float kListMost = 0.92f * kListCap;     // ... and at most about that many (by a sample of a quarter)
// Up to that many rows lists reach further down: a longer list costs 1 to 2 us there, a row that looks again 13.  Without / with,
// us, 128256 logits at top-p 0.9: falling by 4 over the vocabulary, 8 rows 34.3 / 21.7, 64 38.6 / 26.7, 256 55.7 / 44.2; rows
// without a trend 20.8 / 21.7, 25.1 / 26.8, 42.8 / 44.5.  With more rows a CU has others to work on meanwhile: 1024 rows that
// fall 161 / 142 (184 before the lists), without a trend 135 / 140.
constexpr unsigned kFewRows = 256;

// What bounds it: the loads (1024 x 128256 logits, 525 MB: greedy rows 80 us, 6.5 TB/s, rows without a cut 86, with one 95 to 100),
// as long as enough wavefronts are there to compute while others wait: 64 registers and 36 KB of LDS let four workgroups share
// a CU (122 registers and two workgroups before, 143 us; three: 114).  For that the pass keeps no more alive than the
// slice and a few sums, bins a quarter of the elements (all of them took an LDS atomic and nine vector instructions each,
// with the slice's mass as their sum; the exponentials of all take eight), lists without ballots (a lane writes
// what it finds into a strip of its own), and looks all places of the window up at once, a lane each.
template <bool STREAM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void sampler_scan_kernel(SamplerParams sp, char* ws, int slices, int slice_elems)
{
    __shared__ ScanLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long r = blockIdx.x / slices;
    const int slice = blockIdx.x % slices;
    const float* __restrict__ x = sp.logits + r * sp.stride;
    const SliceRange g = slice_range(slice, slice_elems, (int)sp.vocab);
    const RowWs W = row_ws(ws, r, slices);
    const float T = sp.temperature[r];
    const bool greedy = (T == 0.f);
    const float top_p = sp.top_p[r];
    // rows with a min-p or top-k filter are finished from their lists alone, whatever top_p is
    const int top_k = sp.top_k ? sp.top_k[r] : 0;
    const float min_p = sp.min_p ? sp.min_p[r] : 0.f;
    const bool filtered = top_k > 0 || min_p > 0.f;
    const bool cut = !greedy && (top_p < 1.f || filtered);

    float xv[32];
    SPD_LOAD_SLICE(STREAM, xv, x, g, tid)
    if (tid < kGuessBins)
        L.hist[tid] = 0u;
    if (tid == 0)
        L.emitted = 0u;
    lds_barrier();
    // a shorter slice fills fewer registers: only those are looked at (1024 x 4096 35.2 -> 27.5 us, 64 x 32000
    // 21.0 -> 18.3)
    const int steps = (g.e1 - g.e0 + kIter - 1) / kIter;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j >= steps)
            break;
        if (g.e0 + (j + 1) * kIter > g.e1)  // the slice ends in here
            mask_four(xv[4 * j], xv[4 * j + 1], xv[4 * j + 2], xv[4 * j + 3], g.e0 + j * kIter + tid * 4 - (g.e1 - 4));
#pragma unroll
        for (int k = 0; k < 4; k += 2)
            mx = fmaxf(fmaxf(mx, xv[4 * j + k]), xv[4 * j + k + 1]);
    }
    mx = wave_max_f32(mx);
    if (lane == 0)
        L.red_f[wave] = mx;
    lds_barrier();
    mx = L.red_f[0];
    for (int w = 1; w < kWaves; ++w)
        mx = fmaxf(mx, L.red_f[w]);
    mx = uniform(mx);

    if (greedy) {
        int mi = 0x7fffffff;
#pragma unroll
        for (int q = 31; q >= 0; --q)
            if (q < 4 * steps && xv[q] == mx)
                mi = g.e0 + (q >> 2) * kIter + tid * 4 + (q & 3);
        for (int o = 32; o > 0; o >>= 1)
            mi = min(mi, __shfl_xor(mi, o));
        if (lane == 0)
            L.red_i[wave] = mi;
        lds_barrier();
        if (tid == 0) {
            for (int w = 0; w < kWaves; ++w)
                mi = min(mi, L.red_i[w]);
            SliceStat* st = stat_at(W, slice);
            st->max_x = mx;
            st->argmax = mi;
        }
        return;
    }

    // ---- mass of the slice relative to its maximum.  The constant is cut in two so that the second part is
    // positive: a logit of -inf then meets no infinities of opposite sign.  Every fourth element is counted by its bin,
    // counted down from the maximum; what lies past the last is not. ----
    const RowConst rc = row_const(T);
    float c_hi = rc.c_hi, c_lo = rc.c_lo;
    if (c_lo <= 0.f) {
        c_hi = __uint_as_float(__float_as_uint(c_hi) - (c_hi > 0.f ? 1u : 0u));
        c_lo = (float)(rc.cd - (double)c_hi);
    }
    c_hi = uniform(fmaxf(c_hi, 1.2e-38f));
    c_lo = uniform(fmaxf(c_lo, 1.2e-38f));
    const float ref = mx == -INFINITY ? 0.f : mx, down16 = uniform(-16.f * c_hi);
    double m = 0.0;
    float squares = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j >= steps)
            break;
        float s4 = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float d = xv[4 * j + k] - ref;
            // (a logit that is not a number: zero, as in prob(); 0 .. 1 is a modifier of the instruction and costs nothing)
            const float p = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(__builtin_fmaf(d, c_hi, d * c_lo)), 0.f, 1.f);
            s4 += p;
            squares = __builtin_fmaf(p, p, squares);
            if (k == (j & 3) && cut) {
                const unsigned off = (unsigned)(d * down16);  // sixteenths of an octave
                if (off < 4u * kGuessBins)
                    atomicAdd((unsigned*)((char*)L.hist + (off & ~3u)), 1u);
            }
        }
        m += (double)s4;
        if (j & 1)
            __builtin_amdgcn_sched_barrier(0);
    }
    m = wave_scan_f64(m);
    squares = wave_scan_f32(squares);
    if (lane == 63) {
        L.mass[wave] = m;
        L.squares[wave] = squares;
    }
    lds_barrier();
    if (wave == 0) {
        double S = 0.0;
        float sq = 0.f;
        for (int w = 0; w < kWaves; ++w) {
            S += L.mass[w];
            sq += L.squares[w];
        }
        float x_lo = INFINITY, x_hi = INFINITY, x_cut = 0.f;
        if (cut) {
            const uint4 q4 = *reinterpret_cast<const uint4*>(&L.hist[4 * lane]);
            float own = (float)(q4.x + q4.y + q4.z + q4.w), before = wave_scan_f32(own) - own;
            L.cum[4 * lane] = before;
            L.cum[4 * lane + 1] = before + (float)q4.x;
            L.cum[4 * lane + 2] = before + (float)(q4.x + q4.y);
            L.cum[4 * lane + 3] = before + (float)(q4.x + q4.y + q4.z);
            if (lane == 63)
                L.cum[kGuessBins] = before + own;
            // mass by bin, in LDS too
            const float at = __builtin_amdgcn_exp2f(-(float)lane - 0.125f);
            own = at * ((float)q4.x + 0.84089642f * (float)q4.y + 0.70710678f * (float)q4.z + 0.59460356f * (float)q4.w);
            const float all = wave_scan_f32(own);
            before = all - own;
            L.below[4 * lane] = before;
            L.below[4 * lane + 1] = before += at * (float)q4.x;
            L.below[4 * lane + 2] = before += at * 0.84089642f * (float)q4.y;
            L.below[4 * lane + 3] = before += at * 0.70710678f * (float)q4.z;
            if (lane == 63)
                L.below[kGuessBins] = all;
            const float m_all = uniform(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(all), 63)));
            // The places wanted, lane by lane: the first with more than `n` above it, by mass (lanes 0 to 2) or by count.
            // The row's cut lies where the mass below is 1 - top_p of the row's, and this slice's share of the row is not
            // known: one logit that holds much of its mass has none like it in the other slices, and they may have ones
            // that it has not.  So the window reaches from where the cut would lie if the shares were twice this slice's
            // mass and more to where it would if they were less by twice the spread of its mass, down to 0.15 of it (fixed margins of
            // 1200 logits at least and an octave past the place: as few misses, but 18 us more for 1024 rows at 0.7).  Rows of 128256
            // logits that have to look again (kFewRows rows or less / more), sigma 3: none of 4096 at top-p 0.9 to 0.98, one in 350 at 0.999;
            // with fifty boosted tokens none at 0.95, one in 300 at 0.98, one in three at 0.99; falling by 4 over the vocabulary none /
            // half at 0.9, one in 18 / four in five at 0.95; sigma 1 with boosted tokens nearly all.
            const float per_slice = (float)S - 1.f + 1.f / (float)slices, spread = __builtin_amdgcn_sqrtf(fmaxf(sq - 1.f, 0.f));
            const float q = 0.25f * (1.f - top_p);
            float n = m_all - q * per_slice;
            n = lane == 1 ? m_all - q * fmaxf(per_slice - 2.f * spread, 0.15f * per_slice) : n;
            n = lane == 2 ? m_all - q * (per_slice * 2.f + 4.f + 8.f * spread) : n;
            n = lane == 3 ? m_all - 0.5f * q * per_slice : n;
            n = lane == 4 ? 0.25f * kListLeast : n;
            n = lane == 5 ? 0.25f * kListMost : n;
            // (all k may lie in one slice: a quarter of them are in the sample, 0.43 sqrt(k) more or less, and four times that)
            n = lane == 6 ? fminf(0.25f * (float)top_k + 1.75f * __builtin_amdgcn_sqrtf((float)max(top_k, 0)) + 4.f, 1.0e6f) : n;
            const float* const table = lane < 4 ? L.below : L.cum;
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            int b = 0;  // the last place with no more than n above it (tables begin with 0 and never fall)
#pragma unroll 1
            for (int half = kGuessBins / 2; half > 0; half >>= 1)
                b += table[b + half] <= n ? half : 0;
            const float lo_at = table[b], hi_at = table[b + 1];
            const float z = n >= table[kGuessBins] ? (float)kGuessBins : (float)b + (hi_at > lo_at ? fminf(fmaxf((n - lo_at) * __builtin_amdgcn_rcpf(hi_at - lo_at), 0.f), 1.f) : 0.f);
            auto place = [&](int l) __attribute__((always_inline)) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(z), l)); };
            float z_lo, z_hi = 0.f;
            if (filtered) {
                // as far as the filters can reach
                z_lo = top_k > 0 ? place(6) : (float)kGuessBins;
                if (min_p > 0.f)
                    z_lo = fminf(z_lo, -4.f * __builtin_amdgcn_logf(min_p) + 0.01f);
                z_lo = fminf(z_lo, place(5));
            } else {
                auto upto = [&](float zz) __attribute__((always_inline)) {
                    zz = fminf(fmaxf(zz, 0.f), (float)kGuessBins - 0.001f);
                    const int i = (int)zz;
                    return L.cum[i] + (L.cum[i + 1] - L.cum[i]) * (zz - (float)i);
                };
                // (few logits below the cut, as with a top-p next to 1: their mass says little about where the row's cut lies, and
                // all of them fit)
                const float z_cut = place(0), most = 0.25f * kListMost, at_cut = upto(z_cut);
                const float z_far = L.cum[kGuessBins] - at_cut <= 0.25f * most ? (float)kGuessBins : place(1) + 1.f;
                // (at one row a CU the slowest row is the call, and one that looks again takes 13 us more: lists from the top reach to half
                // of the slice's own mass below the cut, which rows that fall or rise over the vocabulary need)
                const float z_deep = gridDim.x <= kFewRows * (unsigned)slices ? fmaxf(z_far, place(3)) : z_far;
                z_lo = fminf(fmaxf(z_deep, place(4)), place(5));
                if (z_far > place(5)) {
                    // Not from the top: around the place, moving each end towards it until what lies between fits half of the
                    // list, or what the other end leaves of it (lane l tries (l + 1) / 64 of the way).
                    z_hi = fmaxf(place(2) - 1.f, 0.f);
                    const float f = (float)(lane + 1) * (1.f / 64.f);
                    const float under = upto(z_cut + (z_far - z_cut) * f) - at_cut, over = at_cut - upto(z_cut - (z_cut - z_hi) * f);
                    auto last = [&](float v) __attribute__((always_inline)) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); };
                    auto widest = [&](bool fits) __attribute__((always_inline)) {
                        const unsigned long long fit = __ballot(fits);
                        return (float)(~fit ? __ffsll((long long)~fit) - 1 : 64) * (1.f / 64.f);  // (and whatever is narrower)
                    };
                    const float room = fmaxf(0.5f * most, most - last(over));
                    z_lo = z_cut + (z_far - z_cut) * widest(under <= room);
                    z_hi = z_cut - (z_cut - z_hi) * widest(over <= most - fminf(last(under), room));
                }
                x_cut = z_cut;
            }
            const float step = 0.25f * __builtin_amdgcn_rcpf(rc.c_hi);  // a quarter octave
            x_lo = (filtered && z_lo >= (float)kGuessBins && g.e1 - g.e0 <= kListCap) || mx == -INFINITY ? -3.402823466e38f : fmaxf(mx - z_lo * step, -3.402823466e38f);
            x_hi = z_hi <= 0.f ? INFINITY : mx - z_hi * step;
            x_cut = mx - x_cut * step;
        }
        if (lane == 0) {
            L.x_lo = x_lo;
            L.x_hi = x_hi;
            SliceStat* st = stat_at(W, slice);
            st->max_x = mx;
            st->argmax = 0;
            st->mass = S;
            st->x_lo = x_lo;
            st->x_hi = x_hi;
            st->x_cut = x_cut;
        }
    }
    if (!cut)
        return;
    lds_barrier();
    const float x_lo = uniform(L.x_lo), x_hi = uniform(L.x_hi);

    // ---- the list.  Every lane gathers the logits of half of its registers in a strip of its own (a compare, a
    // masked LDS write, a masked addition), then the wavefront copies the strips out one place after another. ----
    float* const out = W.list + (size_t)slice * kListCap;
    auto copy_out = [&](int mine) __attribute__((always_inline)) {
        const int all = (int)__builtin_amdgcn_readlane((int)wave_scan_u32((unsigned)mine), 63);
        if (all == 0)
            return;
        unsigned base = 0u;
        if (lane == 0)
            base = atomicAdd(&L.emitted, (unsigned)all);
        base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
        for (int k = 0; k < kStrip; ++k) {
            const unsigned long long some = __builtin_amdgcn_ballot_w64(mine > k);
            if (some == 0ull)
                break;
            if (mine > k) {
                const unsigned at = __builtin_amdgcn_mbcnt_hi((unsigned)(some >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)some, base));
                if (at < (unsigned)kListCap)
                    out[at] = L.strip[k][tid];
            }
            base += (unsigned)__popcll(some);
        }
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (4 * h >= steps)
            break;
        unsigned pos = 4u * (unsigned)tid;  // byte offset of this lane's next place
        if (x_hi == INFINITY) {
#pragma unroll
            for (int q = 16 * h; q < 16 * h + 16; ++q) {
                if (q % 4 == 0 && q >= 4 * steps)
                    break;
                if (xv[q] >= x_lo) {
                    *(float*)((char*)L.strip + pos) = xv[q];
                    pos += 4u * kBlock;
                }
            }
        } else {
#pragma unroll
            for (int q = 16 * h; q < 16 * h + 16; ++q) {
                if (q % 4 == 0 && q >= 4 * steps)
                    break;
                if (xv[q] >= x_lo && xv[q] < x_hi) {
                    *(float*)((char*)L.strip + pos) = xv[q];
                    pos += 4u * kBlock;
                }
            }
        }
        copy_out((int)(pos / (4u * kBlock)));
    }
    // ---- mass above the window ----
    if (x_hi != INFINITY) {
        RowScale rs;
        rs.max_x = mx;
        rs.c_hi = rc.c_hi;
        rs.c_lo = rc.c_lo;
        double part = 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (j >= steps)
                break;
            float s4 = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                s4 += xv[4 * j + k] >= x_hi ? prob(xv[4 * j + k], rs) : 0.f;
            part += (double)s4;
        }
        part = wave_scan_f64(part);
        if (lane == 63)
            L.mass[wave] = part;
    }
    lds_barrier();
    if (tid == 0) {
        SliceStat* st = stat_at(W, slice);
        double above = 0.0;
        if (x_hi != INFINITY)
            for (int w = 0; w < kWaves; ++w)
                above += L.mass[w];
        st->above = above;
        st->count = L.emitted <= (unsigned)kListCap ? (int)L.emitted : -1;
    }
}

// ---- bin selection by the workgroup ------------------------------------------------------------------
// What the wavefronts tell each other.
struct PickLds {
    double sum[kWaves];
    int bin[2][kWaves];
};

struct BinPick {
    int lo, hi;    // the first bins whose cumulative mass reaches `need_lo` and `need_hi` (kBins: none)
    double total;  // with what lies above the bins
};

// H: the masses of kBins bins in units of `unit`, bin 0 = most probable, complete (a barrier behind the last addition); thread t looks at bins
// 4 t .. 4 t + 3.  Every thread returns the same result.  Two barriers; H may be overwritten and `P` used again once every
// thread has passed another one.
__device__ __forceinline__ BinPick block_pick(const unsigned* H, double unit, double above, double need_lo, double need_hi, PickLds& P)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    static_assert(kBinsPerThread == 4, "one 16-byte read per thread");
    const uint4 q = *reinterpret_cast<const uint4*>(H + 4 * tid);
    const double h[4] = {(double)q.x * unit, (double)q.y * unit, (double)q.z * unit, (double)q.w * unit};
    const double own = (h[0] + h[1]) + (h[2] + h[3]);
    const double incl = wave_scan_f64(own);
    if (lane == 63)
        P.sum[wave] = incl;
    lds_barrier();
    double cum = above + (incl - own), total = above;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        total += P.sum[w];
        cum += w < wave ? P.sum[w] : 0.0;
    }
    int lo = kBins, hi = kBins;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        cum += h[k];
        lo = lo == kBins && cum >= need_lo ? 4 * tid + k : lo;
        hi = hi == kBins && cum >= need_hi ? 4 * tid + k : hi;
    }
    lo = (int)wave_min_u32((unsigned)lo);
    hi = (int)wave_min_u32((unsigned)hi);
    if (lane == 0) {
        P.bin[0][wave] = lo;
        P.bin[1][wave] = hi;
    }
    lds_barrier();
    BinPick r;
    r.lo = r.hi = kBins;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        r.lo = min(r.lo, P.bin[0][w]);
        r.hi = min(r.hi, P.bin[1][w]);
    }
    r.total = total;
    return r;
}

// Folds eight per-lane partial sums (one per 256-element segment j of the wavefront's pass) across the
// wavefront: after the exchange across 32 lanes each half keeps four segments, then two, then one,
// so that lanes 8 s .. 8 s + 7 end up with the sum of segment s (10 exchanges instead of 48).
__device__ __forceinline__ double fold_segments(const float (&s_seg)[8])
{
    const int lane = threadIdx.x & 63;
    const bool up32 = (lane & 32) != 0, up16 = (lane & 16) != 0, up8 = (lane & 8) != 0;
    double a4[4], a2[2], a1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float keep = up32 ? s_seg[4 + j] : s_seg[j];
        const float give = up32 ? s_seg[j] : s_seg[4 + j];
        a4[j] = (double)keep + (double)__shfl_xor(give, 32);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const double keep = up16 ? a4[2 + j] : a4[j];
        const double give = up16 ? a4[j] : a4[2 + j];
        a2[j] = keep + __shfl_xor(give, 16);
    }
    {
        const double keep = up8 ? a2[1] : a2[0];
        const double give = up8 ? a2[0] : a2[1];
        a1 = keep + __shfl_xor(give, 8);
    }
    a1 += __shfl_xor(a1, 4);
    a1 += __shfl_xor(a1, 2);
    a1 += __shfl_xor(a1, 1);
    return a1;
}

// ---- kernel 2: the row-level step ---------------------------------------------------------------------
constexpr int kDirect = kBlock;  // logits told apart directly, one per thread

struct FinishLds {
    union {
        RowLds row;                  // the whole-row routine's
        struct {
            unsigned bins[kBins];    // mass (or elements) by bin
            double seg[kSegPerSlice];
        };
    };
    float2 cand[kDirect];            // the logits that the cut falls among, and what each counts for
    unsigned char cand_slice[kDirect];
    double upper[kDirect];           // sums of what is not below, cut among wavefronts
    PickLds pick;
    double slice_mass[kMaxSlices];   // kept mass of every slice
    double above[kMaxSlices];        // what lies above each slice's window, where it begins, the slice's maximum
    float x_hi[kMaxSlices], max_x[kMaxSlices];
    unsigned cands;
    uint32_t best;
    float lowest[kWaves], highest[kWaves];
};

// One row without (FILTERED = false) or with (true) a min-p / top-k filter, by one workgroup.  False: the
// row has to go to the whole-row routine.
template <bool FILTERED, bool MANY>
__device__ __forceinline__ bool finish_row(const SamplerParams& sp, char* ws, int slices, int slice_elems, FinishLds& L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long r = blockIdx.x;
    const RowWs W = row_ws(ws, r, slices);
    const float* __restrict__ x = sp.logits + r * sp.stride;
    const int V = (int)sp.vocab;
    const float T = sp.temperature[r];
    const float top_p = sp.top_p[r];
    const bool greedy = (T == 0.f);
    const int top_k = FILTERED && sp.top_k ? sp.top_k[r] : 0;
    const float min_p = FILTERED && sp.min_p ? sp.min_p[r] : 0.f;
    const bool cut = !greedy && top_p < 1.f;

    // Lane s of every wavefront holds slice s's statistics (lanes past the last slice repeat it).
    const SliceStat st = *stat_at(W, min(lane, slices - 1));
    const bool mine = lane < slices;
    *reinterpret_cast<uint4*>(L.bins + 4 * tid) = make_uint4(0u, 0u, 0u, 0u);

    const float M = wave_max_f32(st.max_x);
    if (greedy) {
        const unsigned arg = wave_min_u32(st.max_x == M ? (unsigned)st.argmax : 0xffffffffu);
        if (tid == 0)
            sp.tokens[r] = arg >= 0x7fffffffu ? 0 : (int)arg;
        return true;
    }
    RowConst rc = row_const(T);
    if ((cut || FILTERED) && rc.cd == 0.0)
        return false;  // an infinite temperature: all tokens tie, whatever their logits are
    rc.c_hi = uniform(rc.c_hi);
    rc.c_lo = uniform(rc.c_lo);
    RowScale rs;
    rs.max_x = M;
    rs.c_hi = rc.c_hi;
    rs.c_lo = rc.c_lo;
    auto of_lane = [&](double d, int l) __attribute__((always_inline)) -> double {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(d), l), __builtin_amdgcn_readlane(__double2loint(d), l));
    };
    const double cd = of_lane(rc.cd, 0);
    auto wave_total = [&](double d) __attribute__((always_inline)) -> double { return of_lane(wave_scan_f64(d), 63); };
    // lane s: what slice s's masses are worth relative to the row's maximum
    const double scale = mine && st.max_x != -INFINITY ? exp2(((double)st.max_x - (double)M) * cd) : 0.0;
    double kept = scale != 0.0 ? st.mass * scale : 0.0;  // lane s: kept mass of slice s
    double S = wave_total(kept);                         // the row's mass
    float x_tau = -INFINITY;                             // kept: x >= x_tau
    if (cut || FILTERED) {
        // (an empty slice lists nothing and lacks nothing)
        const bool some = mine && scale != 0.0;
        unsigned full = (unsigned)__ballot(some && st.count < 0);  // slices that are read again, all of them (bit s)
        const int wps = slices > 4 ? 1 : slices > 2 ? 2 : slices == 2 ? 4 : 8;  // wavefronts per slice
        const int part = wave & (wps - 1), groups = (slices + kWaves - 1) / kWaves;
        // The listed logits, four per lane and step, two steps requested ahead (one where four workgroups share a CU): a slice belongs to one wavefront (to 2,
        // 4, 8 where there are no more than 4, 2, 1 slices).  Then the slices that are read again, by all wavefronts.
        // f(four logits, slice) for every step, end(slice) behind a slice; no barriers inside.
        auto for_all = [&](auto f, auto end) __attribute__((always_inline)) {
            constexpr int kAhead = MANY ? 1 : 2;
            unsigned left = full;
            for (int n = 0; n < groups + __popc(full); ++n) {
                int s, first, step, count;
                const float* from;
                if (n < groups) {
                    s = n * kWaves + wave / wps;
                    count = s < slices && !((full >> s) & 1u) ? __builtin_amdgcn_readlane(st.count, s) : 0;
                    from = W.list + (size_t)s * kListCap;
                    first = part * 64;
                    step = 64 * wps;
                } else {
                    s = __ffs((int)left) - 1;
                    left &= left - 1u;
                    const SliceRange g = slice_range(s, slice_elems, V);
                    count = g.e1 - g.e0;
                    from = x + g.e0;
                    first = wave * 64;
                    step = kBlock;
                }
                if (4 * first >= count)
                    continue;
                // (byte offsets from `from`: one of the lane's own, the steps' are uniform)
                const unsigned last = 4u * (unsigned)((n < groups ? kListCap : count) - 4), stride = 16u * (unsigned)step;
                unsigned own = 16u * (unsigned)(first + lane);
                auto request = [&](unsigned at, float4 (&v)[kAhead]) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u)
                        v[u] = load4<false>(reinterpret_cast<const float*>(reinterpret_cast<const char*>(from) + min(at + (unsigned)u * stride, last)));
                };
                float4 now[kAhead], next[kAhead];
                request(own, now);
#pragma unroll 1
                for (int i = first; 4 * i < count; i += kAhead * step) {
                    request(own + (unsigned)kAhead * stride, next);
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const int at = 4 * (i + u * step);
                        if (at >= count)
                            break;
                        float v[4] = {now[u].x, now[u].y, now[u].z, now[u].w};
                        if (at + 256 > count) {
                            const int mine4 = (int)((own + (unsigned)u * stride) >> 2);
                            if (n >= groups)
                                mask_four(v[0], v[1], v[2], v[3], mine4 - (count - 4));
                            else
#pragma unroll
                                for (int k = 0; k < 4; ++k)
                                    v[k] = mine4 + k < count ? v[k] : -INFINITY;
                        }
                        f(v, s);
                    }
                    own += (unsigned)kAhead * stride;
#pragma unroll
                    for (int u = 0; u < kAhead; ++u)
                        now[u] = next[u];
                }
                end(s);
            }
        };
        float x_above = INFINITY, x_cand = -INFINITY;  // kept for certain: x >= x_above; dropped: x < x_cand
        float x_floor = -INFINITY;  // rows with a filter: the lowest logit that survives it
        bool by_count = false;
        auto weight = [&](float xq) __attribute__((always_inline)) { return FILTERED && by_count ? (prob(xq, rs) >= min_p ? 1.f : 0.f) : prob(xq, rs); };
        const float octave64 = uniform(64.f * __builtin_amdgcn_rcpf(rc.c_hi));  // 64 octaves of p
        // where all lists reach down to, and two octaves above the highest of the slices' own cuts: where the row's is
        // looked for first
        const float reach = fmaxf(wave_max_f32(some && st.count >= 0 ? st.x_lo : -INFINITY), -3.402823466e38f);
        const float start = wave_max_f32(some ? st.x_cut : -INFINITY) + 0.03125f * octave64;
        if (tid < kMaxSlices) {  // (read behind the next barrier)
            L.above[tid] = some && !FILTERED ? st.above * scale : 0.0;
            L.x_hi[tid] = st.x_hi;
            L.max_x[tid] = st.max_x;
        }
        auto per_lane = [&](const float (&a)[kMaxSlices]) __attribute__((always_inline)) {
            int l = lane;
            asm("" : "+v"(l));  // (its address is not kept in a register)
            return a[l & (kMaxSlices - 1)];
        };
        for (int stage = FILTERED && top_k > 0 ? 0 : 1; stage < 2; ++stage) {
            // stage 0 (rows with top-k): the k-th largest logit of what min-p leaves; stage 1: the nucleus cut
            by_count = FILTERED && stage == 0;
            if (FILTERED && stage == 1) {
                // the survivors' mass
                if (top_k <= 0)
                    full |= (unsigned)__ballot(some && st.x_lo > -3.402823466e38f && prob(st.x_lo, rs) >= min_p);
                __syncthreads();
                if (tid < kMaxSlices)
                    L.slice_mass[tid] = 0.0;
                __syncthreads();
                float lowest = INFINITY;
                double mass = 0.0;
                for_all(
                    [&](const float (&v)[4], int) __attribute__((always_inline)) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float p = prob(v[k], rs);
                            const bool keep = v[k] >= x_floor && p >= min_p && p > 0.f;
                            mass += (double)(keep ? p : 0.f);
                            lowest = keep ? fminf(lowest, v[k]) : lowest;
                        }
                    },
                    [&](int s) __attribute__((always_inline)) {
                        mass = wave_scan_f64(mass);
                        if (lane == 63)
                            atomicAdd(&L.slice_mass[s], mass);
                        mass = 0.0;
                    });
                lowest = -wave_max_f32(-lowest);
                if (lane == 63)
                    L.lowest[wave] = lowest;
                __syncthreads();
                kept = mine ? L.slice_mass[lane] : 0.0;
                S = wave_total(kept);
                for (int w = 0; w < kWaves; ++w)
                    lowest = fminf(lowest, L.lowest[w]);
                x_floor = x_tau = uniform(lowest);
                if (!cut)
                    break;
                __syncthreads();
            }
            const double need = of_lane(by_count ? (double)top_k : (double)here(top_p) * S, 0);  // (in scalar registers)
            // Steps that narrow [x_cand, x_above) down: bin what lies there, find the bins that take the running mass across
            // `need`, sum up what lies above them and list what lies in them.  One is enough, but for many equal or
            // nearly equal logits, and where a window does not reach around the bins.
            double above = 0.0;
            float binned = uniform((float)S), next_binned = binned;  // what a step bins, about
            int n = 0;
            bool equal = false, all = false, open = false;  // (of the candidates; there are no k logits; see below)
            uint32_t tie = 0u;                // equal candidates: their key, if the threshold lies there
            int rounds = 0;
            x_above = INFINITY;
            x_cand = reach;
            float from = start;               // where the first step's bins begin
            auto again = [&](unsigned lacking, float high, float low) __attribute__((always_inline)) {
                // once more, with all logits of those slices, between these two first
                full |= lacking;
                ++rounds;
                above = 0.0;
                binned = uniform((float)S);
                x_above = INFINITY;
                from = FILTERED ? INFINITY : uniform(high);
                x_cand = FILTERED ? -3.402823466e38f : uniform(low);
            };
            for (int tries = 0;; ++tries) {
                if (!equal) {
                    const float top = fminf(tries == 0 ? from : x_above, M);
                    const float range = uniform(fminf(fmaxf(top - x_cand, 1e-30f), (tries > 1 ? 256.f : 1.f) * octave64));
                    const float per = uniform(-(float)kBins * __builtin_amdgcn_rcpf(range)), width = range * (1.f / (float)kBins);  // bins (counted down)
                    // a unit is 2^-31 of what is binned, rounded up to a power of two (no bin overflows), but for the rounding of
                    // its logarithm
                    const int power = ((__float_as_int(binned) >> 23) & 0xff) - 126;
                    const double log_exact = (double)(31 - power) + ((double)top - (double)here(M)) * here(cd);
                    const float log_unit = uniform((float)log_exact);
                    const double unit = by_count ? 1.0 : of_lane(ldexp(1.0 + 0.6931471805599453 * (log_exact - (double)log_unit), power - 31), 0);
                    if (tid == 0) {
                        L.cands = 0u;
                        L.best = 0u;
                    }
                    lds_barrier();  // (the bins are cleared)
                    unsigned upper = 0u, beyond = 0u;  // what lies above the bins, and (counts) past the last
                    for_all(
                        [&](const float (&v)[4], int) __attribute__((always_inline)) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                const float d = v[k] - top, bin = d * per;
                                unsigned w = (unsigned)(__builtin_amdgcn_exp2f(__builtin_fmaf(d, rc.c_hi, log_unit)) + 0.5f);
                                if (FILTERED) {
                                    if (by_count)
                                        w = v[k] > -INFINITY && weight(v[k]) > 0.f ? 1u : 0u;
                                    w = v[k] >= x_floor ? w : 0u;
                                }
                                if (tries > 0)  // (what lies above is in `above` by then)
                                    w = v[k] < x_above ? w : 0u;
                                upper += d > 0.f ? w : 0u;
                                if (FILTERED)
                                    beyond += by_count && bin >= (float)kBins ? w : 0u;
                                if (d <= 0.f && bin < (float)kBins)
                                    atomicAdd(&L.bins[(unsigned)bin], w);
                            }
                        },
                        [](int) {});
                    // (what lies above a window counts from its edge on)
                    if (!FILTERED && tries == 0 && tid < kMaxSlices && !((full >> lane) & 1u)) {
                        const double above_s = L.above[tid];
                        const float bin = fmaxf((L.x_hi[tid] - top) * per, 0.f);
                        if (above_s > 0.0 && bin < (float)kBins)
                            atomicAdd(&L.bins[(unsigned)bin], (unsigned)(above_s / unit));
                    }
                    upper = wave_reduce_u32(upper, 0u, [](unsigned a, unsigned b) { return a + b; });
                    if (lane == 0 && upper)
                        atomicAdd(&L.bins[0], upper);
                    if (FILTERED && by_count) {  // the last bin has no end: the k-th may lie further down than bins reach
                        beyond = wave_reduce_u32(beyond, 0u, [](unsigned a, unsigned b) { return a + b; });
                        if (lane == 0 && beyond)
                            atomicAdd(&L.bins[kBins - 1], beyond);
                    }
                    lds_barrier();
                    // (the bins' masses are good to 1e-6 of what is binned; a miss is noticed below)
                    const double tol = of_lane(by_count ? 0.5 : ldexp((double)binned, -19), 0);
                    const BinPick e = block_pick(L.bins, unit, above, need - tol, by_count ? need - tol : need + tol, L.pick);
                    const double total = of_lane(e.total, 0);
                    const int lo = __builtin_amdgcn_readfirstlane(e.lo);
                    const int hi = by_count && e.hi == kBins - 1 ? kBins : __builtin_amdgcn_readfirstlane(e.hi);
                    // (wider by the rounding of all this: of a bin's number, which grows with its distance from the top, and of the edges,
                    // by what the logits there are rounded to, whatever the maximum is; an edge that fell on the value of a
                    // tie would count all of it as above)
                    const float slack = 4e-3f * width + 4e-7f * fmaxf(fabsf(top), fabsf(top - range)), below_bins = tries > 0 ? x_cand : -3.402823466e38f;
                    const float next_above = lo <= 0 ? x_above : fminf(x_above, top - (float)lo * width + slack);
                    // `need` may lie among the bins' last or below all of them, for all that they can tell (top-p within 2e-6 of 1): the
                    // next step bins what is left from lo down, with as much finer a unit
                    open = !by_count && lo < kBins && hi >= kBins;
                    x_cand = uniform(open ? x_cand : hi >= kBins ? below_bins : fmaxf(below_bins, top - (float)(hi + 1) * width - slack));
                    x_above = uniform(next_above);
                    if (open) {  // (from where all windows begin, if they do below: what lies above is known as a sum)
                        const float begin = -wave_max_f32(some && !((full >> lane) & 1u) && per_lane(L.max_x) >= x_cand ? -per_lane(L.x_hi) : -INFINITY);
                        x_above = uniform(begin > x_cand ? fminf(x_above, begin) : x_above);
                    }
                    // does every slice's window reach around them?  (rows with a filter: all survivors are listed)
                    if (!(FILTERED && !by_count)) {
                        // (what is listed reaches `need` nowhere: the cut lies below some windows.  How far follows from the mass that is
                        // left there, over what the cut leaves: it falls by half an octave in one at least, but in the flattest rows)
                        const bool deeper = !FILTERED && hi >= kBins && !open && rounds < 4;
                        if (deeper) {
                            const float left = 1.f + (float)(need - total) / fmaxf((float)(S - need), 1e-30f);
                            x_cand = uniform(fmaxf(x_above - octave64 * (0.03125f * (float)(1 << rounds)) * (0.25f + __builtin_amdgcn_logf(left)), -3.402823466e38f));
                        }
                        const bool below = st.x_lo <= x_cand || (by_count && prob(st.x_lo, rs) < min_p);
                        // (a slice that lies below all of it has nothing to tell, whatever it listed)
                        const unsigned lacking = (unsigned)__ballot(some && per_lane(L.max_x) >= x_cand && !(below && per_lane(L.x_hi) >= x_above)) & ~full;
                        if (lacking != 0u || deeper) {
                            // (where it lies above a window: what lies above that one counted from its edge on, so that the cut lies here
                            // or higher, and windows that end just above it are no help either)
                            const float near = x_above + octave64 * (0.015625f * (float)(1 << min(rounds, 4)));
                            const bool over = !FILTERED && ((unsigned)__ballot(some && per_lane(L.x_hi) < x_above) & lacking) != 0u;
                            const unsigned more = over ? (unsigned)__ballot(some && per_lane(L.max_x) >= x_cand && per_lane(L.x_hi) < near) & ~full : 0u;
                            again(lacking | more, open ? INFINITY : over ? fmaxf(start, x_above + 0.0625f * octave64) : x_above + 0.004f * octave64, open ? -3.402823466e38f : x_cand);
                            tries = -1;
                            *reinterpret_cast<uint4*>(L.bins + 4 * tid) = make_uint4(0u, 0u, 0u, 0u);
                            continue;
                        }
                    }
                    if (!by_count) {  // what the bins from lo to hi hold: all that another step bins
                        unsigned inside = 0u;
                        for (int b = max(lo, 0) + lane; b <= min(hi, kBins - 1); b += 64)
                            inside += L.bins[b];
                        inside = wave_reduce_u32(inside, 0u, [](unsigned a, unsigned b) { return a + b; });
                        // (without an end: and what lies beyond the bins, with the rounding of them all)
                        const float past = hi >= kBins ? fabsf(binned - (float)(total - above)) + 4e-6f * binned : 0.f;
                        next_binned = uniform(1.001f * ((float)((double)inside * unit) + past) + 1e-30f);
                        lds_barrier();
                    }
                    *reinterpret_cast<uint4*>(L.bins + 4 * tid) = make_uint4(0u, 0u, 0u, 0u);
                    if (by_count && total < need - tol) {
                        if (tries > 0)
                            return false;  // (there were k when all of them were counted)
                        all = true;        // there are no k: all of them
                        n = 0;
                        break;
                    }
                }
                if (tid < kMaxSlices)
                    L.slice_mass[tid] = ((full >> lane) & 1u) || L.max_x[tid] < x_above ? 0.0 : L.above[tid];
                lds_barrier();
                double sure = 0.0;
                float least = INFINITY, most = -INFINITY;  // of the candidates
                for_all(
                    [&](const float (&v)[4], int s) __attribute__((always_inline)) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const float xq = FILTERED && !(v[k] >= x_floor) ? -INFINITY : v[k], w = weight(xq);
                            sure += (double)(xq >= x_above ? w : 0.f);
                            if (xq >= x_cand && xq < x_above) {
                                least = fminf(least, xq);
                                most = fmaxf(most, xq);
                                const unsigned at = atomicAdd(&L.cands, 1u);
                                if (at < (unsigned)kDirect) {
                                    L.cand[at] = make_float2(xq, w);
                                    L.cand_slice[at] = (unsigned char)s;
                                }
                            }
                        }
                    },
                    [&](int s) __attribute__((always_inline)) {
                        sure = wave_scan_f64(sure);
                        if (lane == 63)
                            atomicAdd(&L.slice_mass[s], sure);
                        sure = 0.0;
                    });
                lds_barrier();
                kept = mine ? L.slice_mass[lane] : 0.0;
                if (equal)
                    break;
                above = wave_total(kept);
                if (open && above >= need) {  // (the cut lies above some window after all)
                    const unsigned lacking = (unsigned)__ballot(some && per_lane(L.x_hi) < INFINITY) & ~full;
                    if (lacking == 0u)
                        return false;
                    again(lacking, INFINITY, -3.402823466e38f);
                    tries = -1;
                    __syncthreads();
                    continue;
                }
                n = __builtin_amdgcn_readfirstlane((int)L.cands);
                if (n > 64) {
                    least = -wave_max_f32(-least);
                    most = wave_max_f32(most);
                    if (lane == 0) {
                        L.lowest[wave] = least;
                        L.highest[wave] = most;
                    }
                    lds_barrier();
                    for (int w = 0; w < kWaves; ++w) {
                        least = fminf(least, L.lowest[w]);
                        most = fmaxf(most, L.highest[w]);
                    }
                    least = uniform(least);  // (a branch on what the compiler takes to differ from lane to lane costs registers)
                    most = uniform(most);
                    equal = least == most && !(open && above + (double)n * (double)weight(least) < need);
                    if (equal) {
                        // any number of equal ones needs no list: they are the threshold or it was missed.  What each slice
                        // keeps comes from one more pass over the lists where there are more than the list of candidates holds.
                        if (above < need && above + (double)n * (double)weight(least) >= need)
                            tie = order_key(least);
                        if (!tie || by_count || n <= kDirect)
                            break;
                        x_above = least;
                        x_cand = INFINITY;
                        continue;
                    }
                }
                if (n <= kDirect && !open)
                    break;
                if (tries == 3)
                    return false;  // hundreds of nearly equal logits at the cut
                binned = next_binned;
                __syncthreads();
            }
            // ---- the threshold among them: every thread sums what is not below its own (where there are fewer than eight
            // wavefronts' worth, the wavefronts share the sums) ----
            if (!equal) {
                const int share = n <= 64 ? 3 : n <= 128 ? 2 : n <= 256 ? 1 : 0, first = (wave >> share) * 64, part = wave & ((1 << share) - 1);
                if (first < n) {
                    const float own = L.cand[min(first + lane, n - 1)].x;
                    double upper = 0.0;
#pragma unroll 4
                    for (int j = part; j < n; j += 1 << share) {
                        const float2 c = L.cand[j];
                        upper += c.x >= own ? (double)c.y : 0.0;
                    }
                    L.upper[part * (kDirect >> share) + first + lane] = upper;
                }
                lds_barrier();
                if (wave * 64 < n) {
                    const int i = min(tid, n - 1);
                    double upper = above;
                    for (int p = 0; p < 1 << share; ++p)
                        upper += L.upper[p * (kDirect >> share) + i];
                    const uint32_t best = wave_max_u32(upper >= need ? order_key(L.cand[i].x) : 0u);
                    if (lane == 0 && best)
                        atomicMax(&L.best, best);
                }
            }
            lds_barrier();
            const uint32_t best = equal ? tie : L.best;
            // (0: all of them together fall short)
            if (!all && !(best && (equal || above < need)))
                return false;  // the bins missed the threshold
            const float x_cut = uniform(best ? key_value(best) : -INFINITY);
            if (by_count) {
                x_floor = x_cut;
                __syncthreads();
            } else {
                x_tau = x_cut;
                if (n <= kDirect && tid < n && L.cand[tid].x >= x_tau)
                    atomicAdd(&L.slice_mass[L.cand_slice[tid]], (double)L.cand[tid].y);
                lds_barrier();
                kept = mine ? L.slice_mass[lane] : 0.0;
            }
        }
    }
    // ---- the slice that takes the running mass past u Z (rounding may leave the target at the total: then the last
    // one with mass, and its last kept token), and the mass before it ----
    const double inc = wave_scan_f64(kept), target = (double)sp.uniforms[r] * of_lane(inc, 63);
    const unsigned long long past = __ballot(kept > 0.0 && inc > target), any = __ballot(kept > 0.0);
    bool take_last = past == 0ull;
    const int hit = past ? __ffsll((long long)past) - 1 : any ? 63 - __clzll((long long)any) : -1;
    if (hit < 0) {  // (nothing has any mass)
        if (FILTERED)
            return false;
        if (tid == 0)
            sp.tokens[r] = 0;
        return true;
    }
    double before = of_lane(inc - kept, hit);
    // ---- its segments, in vocabulary order ----
    const SliceRange g = slice_range(hit, slice_elems, V);
    float v[32];
    SPD_LOAD_SLICE(false, v, x, g, tid)
    const int steps = (g.e1 - g.e0 + kIter - 1) / kIter;
    float seg[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        seg[j] = 0.f;
        if (j >= steps)
            continue;
        if (g.e0 + (j + 1) * kIter > g.e1)
            mask_four(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3], g.e0 + j * kIter + tid * 4 - (g.e1 - 4));
        float s4 = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[4 * j + k] = v[4 * j + k] >= x_tau ? prob(v[4 * j + k], rs) : 0.f;
            s4 += v[4 * j + k];
        }
        seg[j] = s4;
    }
    const double own = fold_segments(seg);
    if ((lane & 7) == 0)
        L.seg[(lane >> 3) * kWaves + wave] = own;
    lds_barrier();
    const double m = L.seg[lane], inc_seg = before + wave_scan_f64(m);
    const unsigned long long reach = __ballot(m > 0.0 && inc_seg > target), with = __ballot(m > 0.0);
    take_last = take_last || reach == 0ull;
    const int at = take_last ? (with ? 63 - __clzll((long long)with) : 0) : __ffsll((long long)reach) - 1;
    if (wave != (at & (kWaves - 1)))
        return true;
    // ---- one wavefront walks the segment, which it holds ----
    before = of_lane(inc_seg - m, at);
    const int j_at = at / kWaves;
    float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j == j_at) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                p[k] = v[4 * j + k];
        }
    const double s4 = (((double)p[0] + (double)p[1]) + (double)p[2]) + (double)p[3];
    double run = before + (wave_scan_f64(s4) - s4);
    const int base = g.e0 + j_at * kIter + tid * 4;
    int first = 0x7fffffff, last = -1;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (p[k] > 0.f) {
            last = base + k;
            run += (double)p[k];
            if (run > target && first == 0x7fffffff)
                first = base + k;
        }
    first = (int)wave_min_u32((unsigned)first);
    last = (int)wave_max_u32((unsigned)(last + 1)) - 1;
    const int token = first != 0x7fffffff && !take_last ? first : last;
    if (lane == 0)
        sp.tokens[r] = max(token, 0);
    return true;
}

// The row-level step: what a workgroup does with 4000 to 30000 listed logits, one CU's vector instructions (0.1 us for one on each of
// 16000), between a dozen dependent steps.  Phases of a row of 64 x 128256 (clock stamps, us): statistics 0.6, binning the lists
// 4.7 (their loads 1.5 of it), pick 1.2, sums and candidates 3.4, threshold 0.8, the slice of the token 3 to 4, walk 0.4.
// Before, with (logit, index) pairs, whole histograms from the scan kernel, a select by radix over a list of candidates and
// the token's segment from another read of its slice's pairs: 18.9 us (kernel) against 16 for 64 rows, 42 against 30 for 1024.
// 2048 bins over the few octaves between the lists' common end and the slices' own cuts leave a dozen candidates (1/16
// octave each: 170, some thousands in flat rows), so that neither a second level of bins nor a list that could overflow is needed.
// 80 registers and 34 KB of LDS: three workgroups a CU.  With 128, two, and the token's slice requested ahead (by a guess from
// the masses above the bins): 64 rows the same, 300 rows 55 us for 53, 1024 rows 158 for 150.
// What was tried and taken back: 32 logits of each list in registers across the steps (six unrolled passes, 75 KB of code,
// spills: 41 us for 64 rows), bins that add floats (23 us a pass), lists rewritten for the slices whose window missed
// (slower than reading those slices whole: code that runs once is fetched as it runs).
// Sixteen wavefronts a row for few rows: 64 rows 25.1 -> 26.5 us (T 0.7), 300 rows 54 -> 65.
// Whole calls before / now (us, sigma 3 at top-p 0.95 where nothing else is said): 64 x 128256 33.6 -> 30.0, at T 0.7 31.8 -> 22.7,
// 1024 x 128256 (T 0.2 to 1.2) 194 -> 143, 192 x 50257 with filters 43.6 -> 31.2, 64 x 32000 28.8 -> 18.1, 1024 x 4096 40.9 -> 25.8,
// 1024 x 128256 with filters 201 -> 144, 64 x 128256 with a top-k of 50 39.8 -> 28.4, of 20000 609 -> 73, min-p 1e-5 217 -> 46.
// Rows that look again, 64 x 128256: a trend of 10 over the vocabulary 29.6 -> 34.9, fifty boosted tokens over sigma 1 87 -> 109
// (256 rows 401 -> 140), over sigma 2.5 at top-p 0.98 72 -> 95, top-p 0.999 90 -> 79, 0.999999 50 -> 139.  Such a look is two passes over
// all the logits of a slice by one workgroup, vector instructions again (4 us a slice; more loads in flight change nothing).
// ANY = false: no row has a filter.  ANY = true (filter arrays are given): every row takes the routine it
// needs in one launch, so that the two kinds run side by side.  No instantiation uses scratch memory (12 bytes a lane cost
// 1 us): the whole-row routine is inlined (a call would have the arguments copied to memory), what a slice has above its window
// waits in LDS, and the thresholds of a stage are formed in it, in scalar registers.
// MANY: 64 registers instead of 80 and four workgroups a CU, for numbers of rows that take fewer rounds so; only one step of the
// lists requested ahead is what that costs, half a microsecond to two where the rounds are as many.
template <bool ANY, bool MANY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(MANY ? 8 : 6))) void sampler_finish_kernel(SamplerParams sp, char* ws, int slices, int slice_elems)
{
    __shared__ FinishLds L;
    const long long r = blockIdx.x;
    bool done;
    if (ANY && sp.temperature[r] != 0.f && ((sp.top_k && sp.top_k[r] > 0) || (sp.min_p && sp.min_p[r] > 0.f)))
        done = finish_row<true, MANY>(sp, ws, slices, slice_elems, L);
    else
        done = finish_row<false, MANY>(sp, ws, slices, slice_elems, L);
    if (!done) {
        __syncthreads();
        sample_row_from_memory(sp, r, L.row);
    }
}

__global__ __launch_bounds__(kBlock) void sample_rows_kernel(SamplerParams sp)
{
    __shared__ RowLds lds;
    sample_row_from_memory(sp, blockIdx.x, lds);
}

}  // namespace

// Slices per row: enough workgroups to cover the chip, pieces that fit the registers.
int sampler_slices(long long rows, long long vocab)
{
    const long long smin = (vocab + kSliceMax - 1) / kSliceMax;
    if (smin > kMaxSlices)
        return 0;  // whole-row kernel
    // Two workgroups per CU, at most eight slices unless the vocabulary needs more (a wavefront of the row-level
    // step reads one slice's list), and no slice shorter than 4096 logits.
    long long s = (512 + rows - 1) / rows;
    const long long smax_small = vocab / 4096 > 1 ? vocab / 4096 : 1;
    if (s > smax_small) s = smax_small;
    if (s > 8) s = 8;
    if (s < smin) s = smin;
    return (int)s;
}

size_t sampler_workspace_bytes(long long rows, long long vocab)
{
    const int s = sampler_slices(rows, vocab);
    return 256 + (s ? (size_t)rows * sliced_row_bytes(s) : 0);
}

hipError_t launch_sampler(const SamplerParams& p, void* ws, hipStream_t s)
{
    const int slices = sampler_slices(p.rows, p.vocab);
    const bool aligned = (p.stride % 4 == 0) && ((uintptr_t)p.logits % 16 == 0);
    // Short rows that are not aligned take the whole-row kernel, one launch whose passes all hit the L2.  The
    // two sides at 64 rows: 2001 logits 17.7 us against 19.2 in the sliced kernels, 4001 20.8 / 19.8, 5001
    // 22.7 / 19.2; without a cut 4001 9.5 / 10.1, 5001 10.7 / 9.9; with filters 5001 31.9 / 33.0, 7001 38.5 / 33.0;
    // the lines lie within 1000 logits of these from 1 to 2048 rows, except near 768.  (Greedy rows alone
    // would cross at 11000, 4.6 / 5.9 us at 5001: they are not known here.  The sliced side is 1 to 2 us faster since, which moves
    // the lines by some hundred logits.)
    const bool filters = p.top_k || p.min_p;
    const long long least = aligned ? 4 : filters ? 6144 : 4096;
    if (slices == 0 || p.vocab < least) {
        hipLaunchKernelGGL(sample_rows_kernel, dim3((unsigned)p.rows), dim3(kBlock), 0, s, p);
        return hipGetLastError();
    }
    int slice_elems = (int)((p.vocab + slices - 1) / slices);
    slice_elems = (slice_elems + 3) / 4 * 4;
    // Logits that the last-level cache (256 MB) cannot hold are read past it: 1024 x 128256 (525 MB) 207 -> 202 us;
    // 64 x 128256 (33 MB, where the LM head has just left them) would lose, 38.9 / 39.9.
    const bool stream = 4.0 * (double)p.rows * (double)p.vocab >= 256e6;
    hipLaunchKernelGGL(stream ? sampler_scan_kernel<true> : sampler_scan_kernel<false>, dim3((unsigned)(p.rows * slices)), dim3(kBlock), 0, s, p, (char*)ws, slices,
                       slice_elems);
    // Four row-level workgroups a CU (1024 at once) instead of three (768) where that takes fewer rounds; three / four, us a call:
    // 800 x 50256 63.5 / 60.6, 1024 x 128256 153.8 / 145.0, 1024 x 32000 56.4 / 53.8, 4096 x 8192 94.6 / 90.1; as many rounds:
    // 1536 x 50256 106.0 / 108.2, 512 x 128256 81.2 / 82.1.  With filters three (1024 x 128256, top-k 50: 133.1 / 134.4).
    const auto finish = filters                                          ? sampler_finish_kernel<true, false>
                        : (p.rows + 1023) / 1024 < (p.rows + 767) / 768 ? sampler_finish_kernel<false, true>
                                                                         : sampler_finish_kernel<false, false>;
    hipLaunchKernelGGL(finish, dim3((unsigned)p.rows), dim3(kBlock), 0, s, p, (char*)ws, slices, slice_elems);
    return hipGetLastError();
}

}  // namespace spd
