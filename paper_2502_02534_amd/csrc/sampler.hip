// Temperature / nucleus / inverse-CDF token sampler.
//
// Two paths.  The sliced path (below: two stream-ordered kernels) reads a row from HBM once, leaves
// what the row-level step needs in the workspace, and finds the exact nucleus threshold without
// sorting.  The whole-row routine (one workgroup per row, every pass from memory) covers what the
// sliced path does not take: vocabularies of fewer than 4 logits, the rare row whose candidate set
// overflows, rows whose min-p or top-k filter reaches further down than the sliced path's windows, and,
// among rows that do not start on a 16-byte boundary, short ones and those whose positions (up to three
// more than logits) overrun the slices that the vocabulary is cut into (so 16382 to 16384 logits in one slice,
// 131070 to 131072 in eight, 262142 to 262144 in sixteen).
//
// Probabilities are evaluated by one shared routine, p_i = 2^((x_i - max) c) with
// c = log2(e)/T carried as hi + lo floats, so every pass sees the same bits; every sum that
// decides something is carried in fp64; comparisons that define the kept set are on bit
// patterns, so all ties with the threshold are kept by construction.
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
//           registers and leaves behind everything the row-level step can need from it:
//           the slice maximum (and its lowest index), the slice mass relative to that maximum,
//           a histogram of mass over bins of width 1/16 in log2 p (the bin of a logit is
//           floor(x c 16), an integer function of x alone, so a slice histogram differs from
//           the row's by an integer shift; mass is accumulated in u32 fixed point relative to the
//           bin's own reference), and the elements the nucleus cut can fall among, written out as
//           (logit, index) pairs.  Which elements those are is a local guess: the slice finds its
//           own cut bin L from its own histogram; if the slice's elements down to a few bins
//           past L fit the budget it emits from the top (bins 0 .. L + margin, as far as the
//           budget goes), otherwise a window of bins centred on L, as wide as the budget allows,
//           and it sums the mass above the window per 256-element segment.  A slice whose cut bin
//           alone exceeds the budget emits nothing.
//   finish  (rows)  combines the slice maxima and histograms into the row's cut bins [lo, hi].
//           A slice is "covered" if its emitted bins contain [lo, hi] and everything it summed as
//           above its window really is above lo; its emitted elements are then classified with
//           p_i = 2^((x_i - row max) c) exactly as defined (kept for certain, candidate, dropped).
//           Slices that are not covered are read a second time by this workgroup.  The exact
//           threshold is found among the candidates by radix select on the logit's bit pattern
//           with fp64 masses; kept candidates join their segments; the segments are scanned and
//           the walk ends inside the segment that contains u * Z.
//           Rows with a min-p or top-k filter (a second instantiation of the kernel, launched in place
//           of the first when filter arrays are given, takes both kinds of row): the scan kernel writes
//           such a row out from the top as far as the budget goes, and the survivors of the filters,
//           found among the pairs, become the candidate list.
//
// With the row statistics exchanged through memory between two kernels, plain stores and loads do.
// =============================================================================================
constexpr int kIter = kBlock * 4;         // elements one float4 per thread covers
constexpr int kSliceMax = 8 * kIter;      // elements per workgroup: 8 float4 per thread
constexpr int kMaxSlices = 16;
constexpr int kSegPerSlice = kSliceMax / kSeg;  // 64
constexpr int kCandCap = 3072;
constexpr int kPubBins = 1024;    // histogram bins of a slice (64 octaves below its maximum)
constexpr int kEmitCap = 2048;    // (logit, index) pairs a slice may write out
constexpr int kTopProbe = 0;      // a slice emits from the top if its elements down to L + kTopProbe fit
constexpr int kTopMargin = 160;   // ... and then goes on down to L + kTopMargin at most (10 octaves)
static_assert(kMaxSlices * kSegPerSlice <= kMaxSegments, "segment table too small");

struct SliceStat {
    float max_x;
    int argmax;
    double rest;      // estimated mass of the slice's bins past win_hi, in units of 2^(bin_coord(max_x) / 16)
    int win_lo;       // emitted bins [win_lo, win_hi], counted down from the bin of max_x
    int win_hi;
    int count;        // emitted pairs; -1: the slice emitted nothing although the row has a cut
    int pad;
};
static_assert(sizeof(SliceStat) <= 64, "slice statistics are kept 64 bytes apart");

__host__ __device__ inline size_t sliced_row_bytes(int slices)
{
    return (size_t)slices * (64 + (size_t)kPubBins * 4 + (size_t)kSegPerSlice * 8 + (size_t)kEmitCap * 8);
}

struct RowWs {
    char* stat;                // [slices] SliceStat, 64 B apart
    unsigned* hist;            // [slices][kPubBins]
    double* seg;               // [slices][kSegPerSlice] mass above the window (whole mass when nothing is cut)
    unsigned long long* emit;  // [slices][kEmitCap] logit bits | index << 32
};

__device__ __forceinline__ RowWs row_ws(char* base, long long row, int slices)
{
    char* p = base + row * sliced_row_bytes(slices);
    RowWs w;
    w.stat = p;
    p += (size_t)slices * 64;
    w.hist = (unsigned*)p;
    p += (size_t)slices * kPubBins * 4;
    w.seg = (double*)p;
    p += (size_t)slices * kSegPerSlice * 8;
    w.emit = (unsigned long long*)p;
    return w;
}

__device__ __forceinline__ SliceStat* stat_at(const RowWs& w, int s) { return (SliceStat*)(w.stat + (size_t)s * 64); }

// Monotone map of a float onto unsigned integers (larger float -> larger key).
__device__ __forceinline__ uint32_t order_key(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Bin coordinate of a logit: one multiply and a floor, the same in every kernel.
__device__ __forceinline__ float bin_coord(float x, float c16) { return floorf(x * c16); }

// Bin of a logit counted down from the bin of a maximum, clamped to [0, kBins-1].
__device__ __forceinline__ int bin_below(float kf_max, float kf)
{
    return (int)fminf(fmaxf(kf_max - kf, 0.f), (float)(kBins - 1));
}

// A slice's histogram is kept in the workspace as a ring over the bin coordinate itself (bin b of a slice
// whose maximum has coordinate kf goes to place (kf - b) mod kPubBins), so that the row-level kernel can
// request the same place of every slice before it knows any of the maxima.
__device__ __forceinline__ int ring_base(float kf)
{
    // (floats beyond 2^62 are multiples of kPubBins; a slice of -inf holds no units)
    return fabsf(kf) < 4.0e18f ? (int)((long long)kf & (kPubBins - 1)) : 0;
}

struct RowConst {
    float c_hi, c_lo, c16;
    double cd;
};

__device__ __forceinline__ RowConst row_const(float T)
{
    RowConst k;
    k.cd = 1.4426950408889634 / (double)T;
    k.c_hi = (float)k.cd;
    k.c_lo = (float)(k.cd - (double)k.c_hi);
    k.c16 = k.c_hi * 16.f;
    return k;
}

// Mass that one unit of a bin's fixed-point histogram stands for, relative to the reference of
// bin 0: 2^-15 2^(-bin/16) (the root in fp32: an estimate is all that is needed).
__device__ __forceinline__ double bin_unit(int bin)
{
    const double root = (double)__builtin_amdgcn_exp2f(-0.0625f * (float)(bin & 15));
    return root * __hiloint2double((1023 - 15 - (bin >> 4)) << 20, 0);
}

// A row that does not start on a 16-byte boundary (a vocabulary that is not a multiple of 4) is
// handled in positions counted from the boundary before it: position i holds logit i - lead, and
// positions below `lead` hold none.  Everything up to the token (pairs, segments, the walk) is in
// positions.
__device__ __forceinline__ int row_lead(const float* x) { return (int)(((uintptr_t)x >> 2) & 3); }

// Slice [e0, e1) of a row's positions; [v0, v4end) are its whole float4s.
struct SliceRange {
    int e0, e1, v0, v4end, lead;
};

__device__ __forceinline__ SliceRange slice_range(int slice, int slice_elems, int V, int lead)
{
    SliceRange g;
    g.e0 = slice * slice_elems;
    g.e1 = min(V + lead, g.e0 + slice_elems);
    g.v0 = slice == 0 && lead > 0 ? 4 : g.e0;
    g.v4end = g.e1 & ~3;
    g.lead = lead;
    return g;
}

// Loads a slice into 32 registers per thread; `xa` points at position 0.  Every load is unconditional
// (lanes outside the whole float4s re-read the nearest one), so that the hardware's in-order load
// counter stays exact for the compiler and later loads need not wait for these.  SPD_MASK_SLICE,
// applied where the values are first needed, replaces what lies outside the row by -inf and, in a slice that
// begins or ends inside a float4, fetches the logits there.  (Fetched under a branch per float4 they cost
// every slice that is not full about a microsecond, 1024 greedy rows of 1000 logits 11.9 us against 9.6, and
// the row-level kernel some 20 registers.)  Every slice holds at least one
// whole float4 (the host sends rows shorter than that to the whole-row kernel, and slices are never
// shorter than about 2000).
// STREAM: not kept in the caches (the pass of launch_sampler over logits that do not fit them).
template <bool STREAM> __device__ __forceinline__ float4 load4(const float* at)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 v = STREAM ? __builtin_nontemporal_load((const f32x4*)at) : *(const f32x4*)at;
    return make_float4(v[0], v[1], v[2], v[3]);
}

#define SPD_LOAD_SLICE(STREAM, xv, xa, g, tid)                                          \
    _Pragma("unroll") for (int j = 0; j < 8; ++j)                                       \
    {                                                                                   \
        const int i_ = min((g).e0 + j * kIter + (tid) * 4, (g).v4end - 4);              \
        const float4 v_ = load4<STREAM>((xa) + (j == 0 ? max(i_, (g).v0) : i_));        \
        (xv)[4 * j] = v_.x;                                                             \
        (xv)[4 * j + 1] = v_.y;                                                         \
        (xv)[4 * j + 2] = v_.z;                                                         \
        (xv)[4 * j + 3] = v_.w;                                                         \
    }
#define SPD_MASK_SLICE(xv, xa, g, tid)                                                  \
    _Pragma("unroll") for (int j = 0; j < 8; ++j)                                       \
    {                                                                                   \
        const int i_ = (g).e0 + j * kIter + (tid) * 4;                                  \
        if (i_ < (g).v0 || i_ >= (g).v4end)                                             \
            (xv)[4 * j] = (xv)[4 * j + 1] = (xv)[4 * j + 2] = (xv)[4 * j + 3] = -INFINITY; \
    }                                                                                   \
    if ((g).v0 > (g).e0 || (g).e1 > (g).v4end)                                          \
        load_slice_ends(xv, xa, g, tid);

// The logits of the float4s that a slice only partly fills: up to three before its first whole one (thread
// 0), up to three behind its last.
__device__ __forceinline__ void load_slice_ends(float (&xv)[32], const float* __restrict__ xa, const SliceRange& g, int tid)
{
    if (g.v0 > g.e0 && tid == 0) {
#pragma unroll
        for (int k = 1; k < 4; ++k)
            if (k >= g.lead)
                xv[k] = xa[k];
    }
    const int behind = g.v4end - g.e0 - 4 * tid;  // of this thread's first float4
    if (g.e1 > g.v4end && behind >= 0 && behind % kIter == 0) {
        float end[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            end[k] = g.v4end + k < g.e1 ? xa[g.v4end + k] : -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (behind == j * kIter) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    xv[4 * j + k] = end[k];
            }
    }
}

// ---- kernel 1: the pass over the logits --------------------------------------------------------------
constexpr int kWaveStage = kEmitCap / kWaves * 2;  // pairs one wavefront may gather (twice its even share)

struct ScanLds {
    unsigned hist[kPubBins + 64];       // + one place per lane for what lies past the last bin
    unsigned cumq[kPubBins];            // inclusive running sum of hist
    unsigned long long stage[kWaves][kWaveStage + 1];  // each wavefront's pairs, copied out in one piece (+ one
                                                       // place that takes whatever does not fit)
    double wave_mass[kWaves];
    unsigned wave_q[kWaves];
    float red_f[kWaves];
    int red_i[kWaves];
    double rest;               // estimated mass of the bins past the window
    int cut_bin;               // the slice's own cut bin L
    int best;                  // scratch of the window search
    int emitted;               // places reserved in the slice's list so far
    int overflow;              // some wavefront gathered more pairs than it has room for
};

// Barrier between phases that exchange data through LDS only: waits for this wavefront's LDS
// traffic, not for its global loads and stores (a __syncthreads would drain those too, and the
// slice's logits and the published results are still in flight at most barriers of this kernel).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Fixed-point mass of a logit inside its bin: 32768 2^(f/16) for f in [0, 1), as a quadratic in f:
// the series 32768 + a1 f + a2 f^2 + a3 f^3 with f^3 replaced by its best quadratic on [0, 1],
// (48 f^2 - 18 f + 1) / 32 (error a3 / 32 = 0.014 units; the next term of the series is below
// 0.005).  Values run from 32768 to 34219.  NaN (positions past the end of a slice) converts to 0.
// The scan kernel's pass over the logits is bound by its vector instructions (every instruction
// per logit costs it about 2 % of its time), hence the count of every one here and below.
__device__ __forceinline__ unsigned bin_units(float f)
{
    const float a1 = 1419.5653f, a2 = 30.749034f, a3 = 0.44403f;
    const float b0 = 32768.5f + a3 / 32.f, b1 = a1 - a3 * (18.f / 32.f), b2 = a2 + a3 * (48.f / 32.f);
    return (unsigned)__builtin_fmaf(__builtin_fmaf(b2, f, b1), f, b0);
}

// Folds eight per-lane partial sums (one per 256-element segment j of the wavefront's pass) across the
// wavefront: after the exchange across 32 lanes each half keeps four segments, then two, then one,
// so that lane 8 s ends up with the sum of segment s (10 exchanges instead of 48).
__device__ __forceinline__ float fold_segments(const float (&s_seg)[8])
{
    const int lane = threadIdx.x & 63;
    const bool up32 = (lane & 32) != 0, up16 = (lane & 16) != 0, up8 = (lane & 8) != 0;
    float a4[4], a2[2], a1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float keep = up32 ? s_seg[4 + j] : s_seg[j];
        const float give = up32 ? s_seg[j] : s_seg[4 + j];
        a4[j] = keep + __shfl_xor(give, 32);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float keep = up16 ? a4[2 + j] : a4[j];
        const float give = up16 ? a4[j] : a4[2 + j];
        a2[j] = keep + __shfl_xor(give, 16);
    }
    {
        const float keep = up8 ? a2[1] : a2[0];
        const float give = up8 ? a2[0] : a2[1];
        a1 = keep + __shfl_xor(give, 8);
    }
    a1 += __shfl_xor(a1, 4);
    a1 += __shfl_xor(a1, 2);
    a1 += __shfl_xor(a1, 1);
    return a1;  // lanes 8 s .. 8 s + 7 hold segment j = 4 (lane/32) + 2 (lane/16 % 2) + lane/8 % 2 = lane >> 3
}

template <bool STREAM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void sampler_scan_kernel(SamplerParams sp, char* ws, int slices, int slice_elems)
{
    __shared__ ScanLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long r = blockIdx.x / slices;
    const int slice = blockIdx.x % slices;
    const float* __restrict__ row_x = sp.logits + r * sp.stride;
    const int lead = row_lead(row_x);
    const float* __restrict__ x = row_x - lead;  // position 0
    const SliceRange g = slice_range(slice, slice_elems, (int)sp.vocab, lead);
    const RowWs W = row_ws(ws, r, slices);
    const float T = sp.temperature[r];
    const bool greedy = (T == 0.f);
    const float top_p = sp.top_p[r];
    // rows with a min-p or top-k filter are finished from their pairs alone, whatever top_p is
    const bool filtered = (sp.top_k && sp.top_k[r] > 0) || (sp.min_p && sp.min_p[r] > 0.f);
    const bool cut = !greedy && (top_p < 1.f || filtered);

    float xv[32];
    SPD_LOAD_SLICE(STREAM, xv, x, g, tid)
    for (int b = tid; b < kPubBins + 64; b += kBlock)
        L.hist[b] = 0u;
    if (tid == 0) {
        L.cut_bin = kPubBins - 1;
        L.best = -1;
        L.emitted = 0;
        L.overflow = 0;
        L.rest = 0.0;
    }
    // wavefronts whose 32 x 64 x 4 logits all lie inside the row skip the masking of its ends
    const bool whole = g.e0 + 7 * kIter + (tid | 63) * 4 + 4 <= g.v4end && g.e0 + (tid & ~63) * 4 >= g.v0;
    if (!whole) {
        SPD_MASK_SLICE(xv, x, g, tid)
    }
    float mx = -INFINITY;
#pragma unroll
    for (int q = 0; q < 32; ++q)
        mx = fmaxf(mx, xv[q]);
    mx = wave_max_f32(mx);
    if (lane == 0)
        L.red_f[wave] = mx;
    lds_barrier();
    mx = L.red_f[0];
    for (int w = 1; w < kWaves; ++w)
        mx = fmaxf(mx, L.red_f[w]);

    if (greedy) {
        int mi = 0x7fffffff;
#pragma unroll
        for (int q = 31; q >= 0; --q)
            if (xv[q] == mx)
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

    const RowConst rc = row_const(T);
    RowScale rs;
    rs.max_x = mx;
    rs.c_hi = rc.c_hi;
    rs.c_lo = rc.c_lo;
    const float kf_loc = bin_coord(mx, rc.c16);
    unsigned long long* out = W.emit + (size_t)slice * kEmitCap;
    double* seg_out = W.seg + (size_t)slice * kSegPerSlice;

    if (!cut) {
        // ---- nothing is cut: the mass of every 256-element segment, relative to the slice maximum ----
        float s_seg[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            s_seg[j] = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float xq = xv[4 * j + k];
                s_seg[j] += (whole || xq != -INFINITY) ? prob(xq, rs) : 0.f;
            }
        }
        const float a1 = fold_segments(s_seg);
        if ((lane & 7) == 0)
            seg_out[(lane >> 3) * kWaves + wave] = (double)a1;
        if (tid == 0) {
            SliceStat* st = stat_at(W, slice);
            st->max_x = mx;
            st->argmax = 0;
            st->rest = 0.0;
            st->win_lo = 0;
            st->win_hi = -1;
            st->count = 0;
        }
        return;
    }

    // ---- histogram of mass over the slice's own bins.  Elements 64 octaves and more below the slice
    // maximum belong to the last bin; each lane collects them in a place of its own (they would
    // otherwise all meet at one LDS address) and the places are added to the last bin afterwards.
    // Positions past the end of the slice (-inf) land there too, with zero units. ----
    // (byte offsets: four times the bin, formed in floating point, so that one conversion gives
    // the LDS address; what lands between the last bin and the lane's own place belongs to the
    // last bin all the same)
    const float far4 = (float)(4 * (kPubBins + lane)), kf_loc4 = 4.f * kf_loc;
    auto bin_one = [&](float xq) __attribute__((always_inline)) {
        const float t = xq * rc.c16;
        const float kf = floorf(t);
        const float off = fminf(__builtin_fmaf(kf, -4.f, kf_loc4), far4);  // >= 0: kf_loc belongs to the maximum
        atomicAdd((unsigned*)((char*)L.hist + (unsigned)off), bin_units(t - kf));
    };
#pragma unroll
    for (int q = 0; q < 32; ++q)
        bin_one(xv[q]);
    lds_barrier();  // histogram complete
    // what the lanes collected past the last bin belongs to the last bin (every wavefront adds the
    // places up for itself; only the owner of the last bin uses the sum)
    static_assert(kPubBins == 2 * kBlock, "thread t owns bins 2t and 2t+1; the last thread owns the last bin");
    const unsigned far_units = wave_reduce_u32(L.hist[kPubBins + lane], 0u, [](unsigned a, unsigned b) { return a + b; });

    // ---- running sums over the bins (thread t owns bins 2t, 2t+1): fixed-point units for the element
    // counts, estimated mass for the slice's own cut bin ----
    const unsigned q0 = L.hist[2 * tid], q1 = L.hist[2 * tid + 1] + (tid == kBlock - 1 ? far_units : 0u);
    const double m0 = (double)q0 * bin_unit(2 * tid), m1 = (double)q1 * bin_unit(2 * tid + 1);
    unsigned qi = wave_scan_u32(q0 + q1);
    double mi = wave_scan_f64(m0 + m1);
    if (lane == 63) {
        L.wave_q[wave] = qi;
        L.wave_mass[wave] = mi;
    }
    lds_barrier();
    unsigned qbefore = 0u;
    double mbefore = 0.0, mtotal = 0.0;
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) {
            qbefore += L.wave_q[w];
            mbefore += L.wave_mass[w];
        }
        mtotal += L.wave_mass[w];
    }
    qi += qbefore;   // inclusive through bin 2t+1
    mi += mbefore;
    L.cumq[2 * tid] = qi - q1;
    L.cumq[2 * tid + 1] = qi;
    // the one thread whose bins take the running mass across top_p of the total names the cut bin
    const double need = (double)top_p * mtotal;
    if (mi - m0 - m1 < need) {
        if (mi - m1 >= need)
            L.cut_bin = 2 * tid;
        else if (mi >= need)
            L.cut_bin = 2 * tid + 1;
    }
    lds_barrier();
    // ---- which bins to write out.  Element counts come from the fixed-point sums: every element adds
    // between 32768 and 34219 units, so (units >> 15) never undercounts.  Every thread tests two
    // places of the search range; the largest that fits wins. ----
    const int Lb = L.cut_bin;
    auto units = [&](int a, int z) { return L.cumq[z] - (a > 0 ? L.cumq[a - 1] : 0u); };
    auto fits = [&](int a, int z) { return (int)(units(a, z) >> 15) <= kEmitCap; };
    // (a row with a filter: always from the top, as many bins as fit; its filters decide later how
    // far down they reach)
    const bool from_top = filtered || fits(0, min(Lb + kTopProbe, kPubBins - 1));
    int mine = -1;
    if (from_top) {
        // bins 0 .. z, z as large as fits, at most L + kTopMargin
        const int zmax = filtered ? kPubBins - 1 : min(Lb + kTopMargin, kPubBins - 1);
        if (2 * tid + 1 <= zmax && (int)(qi >> 15) <= kEmitCap)
            mine = 2 * tid + 1;
        else if (2 * tid <= zmax && (int)((qi - q1) >> 15) <= kEmitCap)
            mine = 2 * tid;
    } else if (fits(Lb, Lb)) {
        // bins L - w .. L + w, w as large as fits
#pragma unroll
        for (int k = 1; k >= 0; --k) {
            const int w = tid + k * kBlock;
            if (mine < 0 && fits(max(Lb - w, 0), min(Lb + w, kPubBins - 1)))
                mine = w;
        }
    }
    mine = (int)wave_max_u32((unsigned)(mine + 1)) - 1;
    if (lane == 0 && mine >= 0)
        atomicMax(&L.best, mine);
    lds_barrier();
    const int best = L.best;
    int win_lo = 0, win_hi = -1;   // bins written out; win_hi < 0: none
    if (best >= 0) {
        win_lo = from_top ? 0 : max(Lb - best, 0);
        win_hi = from_top ? best : min(Lb + best, kPubBins - 1);
    }
    // the thread that owns bin win_hi knows the estimated mass of everything past it
    if (win_hi >= 0 && (win_hi >> 1) == tid)
        L.rest = mtotal - ((win_hi & 1) ? mi : mi - m1);
    // Bin tests without forming the bin: with t = x c16, bin(x) < a  <=>  floor(t) > kf_loc - a
    // <=>  t >= kf_loc - a + 1 (both sides of the middle inequality are integers); likewise
    // bin(x) <= z  <=>  t >= kf_loc - z, and the last bin takes everything below it (every finite
    // logit: positions past the end of the slice hold -inf and fail the test).
    const float t_above = win_lo <= 0 ? INFINITY : kf_loc - (float)win_lo + 1.f;
    const float t_emit = win_hi < 0 ? INFINITY : (win_hi >= kPubBins - 1 ? -3.0e38f : kf_loc - (float)win_hi);

    // ---- the pairs: every wavefront gathers its own in LDS (the lanes that hold one take consecutive
    // places), reserves as many places in the slice's list and copies them out in one piece ----
    int have = 0;  // pairs this wavefront has gathered (uniform)
    // (one compare, two lane counts that also add the running total, a clamp, the index, the address;
    // logit and index go out of two registers with one two-dword write)
    const unsigned stage_base = (unsigned)(size_t)(__attribute__((address_space(3))) void*)&L.stage[wave][0];
    auto gather = [&](unsigned long long mask /* the wavefront's ballot of pred */, bool pred, float xq,
                      int idx) __attribute__((always_inline)) {
        if (pred) {
            const int pos = min((int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((unsigned)mask, (unsigned)have)),
                                kWaveStage);
            const unsigned addr = stage_base + 8u * (unsigned)pos;
            asm volatile("ds_write2_b32 %0, %1, %2 offset1:1" ::"v"(addr), "v"(xq), "v"(idx) : "memory");
        }
        have += __popcll(mask);
    };
    if (win_hi >= 0) {
        if (win_lo <= 0) {
#pragma unroll
            for (int q = 0; q < 32; ++q) {
                const bool in = xv[q] * rc.c16 >= t_emit;
                gather(__builtin_amdgcn_ballot_w64(in), in, xv[q], g.e0 + (q >> 2) * kIter + tid * 4 + (q & 3));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 32; ++q) {
                const float t = xv[q] * rc.c16;
                const bool in = t >= t_emit, below = t < t_above;  // (two ballots and a scalar AND: no vector work)
                gather(__builtin_amdgcn_ballot_w64(in) & __builtin_amdgcn_ballot_w64(below), in && below, xv[q],
                       g.e0 + (q >> 2) * kIter + tid * 4 + (q & 3));
            }
        }
    }
    int base = 0;
    if (lane == 0 && have) {
        base = atomicAdd(&L.emitted, have);
        if (have > kWaveStage)
            L.overflow = 1;
    }
    base = __builtin_amdgcn_readfirstlane(base);
    lds_barrier();
    // A wavefront that ran out of room (sorted logits can put a slice's whole window into one
    // wavefront) makes the slice publish nothing: the row-level step then reads it a second time.
    const bool publish = win_hi >= 0 && !L.overflow;
    const int total = L.emitted;
    if (tid == 0) {
        SliceStat* st = stat_at(W, slice);
        st->max_x = mx;
        st->argmax = 0;
        st->rest = L.rest;
        st->win_lo = win_lo;
        st->win_hi = publish ? win_hi : -1;
        st->count = publish ? total : -1;
    }
    if (publish)
        for (int i = lane; i < min(have, kWaveStage); i += 64)
            if (base + i < kEmitCap)
                out[base + i] = L.stage[wave][i];
    {
        unsigned* ring = W.hist + (size_t)slice * kPubBins;
        const int place = ring_base(kf_loc) - 2 * tid;
        ring[place & (kPubBins - 1)] = q0;
        ring[(place - 1) & (kPubBins - 1)] = q1;
    }
    // ---- segment sums: what lies above the window (nothing when the window starts at the top) ----
    float a1 = 0.f;
    if (win_hi >= 0 && win_lo > 0) {
        float s_seg[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            s_seg[j] = 0.f;
#pragma unroll
        for (int q = 0; q < 32; ++q)
            if (xv[q] * rc.c16 >= t_above)
                s_seg[q >> 2] += prob(xv[q], rs);
        a1 = fold_segments(s_seg);
    }
    if ((lane & 7) == 0)
        seg_out[(lane >> 3) * kWaves + wave] = (double)a1;
}

// ---- bin selection by the workgroup ------------------------------------------------------------------
struct BinPick {
    int bin;        // first non-empty bin whose cumulative mass reaches `need`
    double above;   // mass strictly above it (including `above0`)
    double in_bin;  // its own mass
    double total;   // sum of the histogram
};

// What the wavefronts tell each other.
struct PickLds {
    double sum[kWaves];
    double above[2][kWaves], in_bin[2][kWaves];  // [0] the first bin that reaches `need`, [1] the last non-empty bin
    int bin[2][kWaves];                          // (-1: none)
};

// H: kBins masses, bin 0 = most probable, in LDS and complete (a barrier behind the last addition); thread
// t owns bins 4 t .. 4 t + 3.  Every thread returns the same result.  With `relative`, `need` is a
// fraction of the histogram's total.  If rounding leaves even the total short of `need`, the last
// non-empty bin is taken (everything is kept).  Two barriers; H may be overwritten and `P` used again once
// every thread has passed another one.
__device__ __forceinline__ BinPick block_pick(const double* H, double above0, double need, bool relative, PickLds& P)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    static_assert(kBinsPerThread == 4, "two 16-byte reads per thread");
    double h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        h[k] = H[4 * tid + k];
    const double own = (h[0] + h[1]) + (h[2] + h[3]);
    const double incl = wave_scan_f64(own);
    if (lane == 63)
        P.sum[wave] = incl;
    lds_barrier();
    double before = above0 + (incl - own), total = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        total += P.sum[w];
        before += w < wave ? P.sum[w] : 0.0;
    }
    if (relative)
        need *= total;
    // this thread's first bin that reaches `need`, and its last non-empty one
    int bin[2] = {-1, -1};
    double above[2] = {0.0, 0.0}, in_bin[2] = {0.0, 0.0}, cum = before;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double next = cum + h[k];
        if (h[k] > 0.0) {
            if (bin[0] < 0 && next >= need) {
                bin[0] = 4 * tid + k;
                above[0] = cum;
                in_bin[0] = h[k];
            }
            bin[1] = 4 * tid + k;
            above[1] = cum;
            in_bin[1] = h[k];
        }
        cum = next;
    }
    const unsigned long long hit = __ballot(bin[0] >= 0), some = __ballot(bin[1] >= 0);
    const int first = hit ? __ffsll((long long)hit) - 1 : -1, last = some ? 63 - __clzll((long long)some) : -1;
    if (lane == (first < 0 ? 0 : first)) {
        P.bin[0][wave] = bin[0];
        P.above[0][wave] = above[0];
        P.in_bin[0][wave] = in_bin[0];
    }
    if (lane == (last < 0 ? 0 : last)) {
        P.bin[1][wave] = bin[1];
        P.above[1][wave] = above[1];
        P.in_bin[1][wave] = in_bin[1];
    }
    lds_barrier();
    // the first wavefront with a hit, else the last one with anything
    int from = -1, kind = 0;
#pragma unroll
    for (int w = kWaves - 1; w >= 0; --w)
        from = P.bin[0][w] >= 0 ? w : from;
    if (from < 0) {
        kind = 1;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            from = P.bin[1][w] >= 0 ? w : from;
    }
    BinPick r;
    r.total = total;
    r.bin = from < 0 ? 0 : P.bin[kind][from];
    r.above = from < 0 ? above0 : P.above[kind][from];
    r.in_bin = from < 0 ? 0.0 : P.in_bin[kind][from];
    return r;
}

// Two block-wide fp64 sums at once (fixed reduction tree).
__device__ void block_sum2_f64(double& a, double& b, double* scratch /* 2 kWaves */)
{
    a = wave_scan_f64(a);
    b = wave_scan_f64(b);
    __syncthreads();
    if ((threadIdx.x & 63) == 63) {
        scratch[threadIdx.x >> 6] = a;
        scratch[kWaves + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    a = 0.0;
    b = 0.0;
    for (int w = 0; w < kWaves; ++w) {
        a += scratch[w];
        b += scratch[kWaves + w];
    }
}

// ---- kernel 2: the row-level step ---------------------------------------------------------------------
struct FinishLds {
    RowLds row;                           // hist / scratch / seg_mass of the row routines
    unsigned long long cand[kCandCap];    // candidates: logit bits | index << 32
    PickLds pick;
    double slice_mass[kMaxSlices];               // kept mass of every slice
    double above[kMaxSlices / kWaves][kWaves];   // what each wavefront found kept for certain among its pairs
    unsigned cand_total;
    unsigned members;                            // candidates in the bin that a select has come down to
    uint32_t kmin[kWaves], kmax[kWaves];
};

// One row without (FILTERED = false) or with (true) a min-p / top-k filter, by one workgroup.  False: the
// row has to go to the whole-row routine.
template <bool FILTERED>
__device__ __forceinline__ bool finish_row(const SamplerParams& sp, char* ws, int slices, int slice_elems, FinishLds& L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long r = blockIdx.x;
    const RowWs W = row_ws(ws, r, slices);
    const float* __restrict__ row_x = sp.logits + r * sp.stride;
    const int lead = row_lead(row_x);
    const float* __restrict__ x = row_x - lead;  // position 0
    const int V = (int)sp.vocab;
    const float T = sp.temperature[r];
    const float top_p = sp.top_p[r];
    const bool greedy = (T == 0.f);
    const int top_k = FILTERED && sp.top_k ? sp.top_k[r] : 0;
    const float min_p = FILTERED && sp.min_p ? sp.min_p[r] : 0.f;
    const bool cut = !greedy && top_p < 1.f;
    const int nseg = slices * kSegPerSlice;
    double* seg_mass = L.row.seg_mass;

    // Lane s of every wavefront holds slice s's statistics (lanes past the last slice repeat it); what all
    // lanes need of a slice is read out of its lane.
    const SliceStat st = *stat_at(W, min(lane, slices - 1));
    const double seg0 = W.seg[min(tid, nseg - 1)];
    if (tid == 0)
        L.cand_total = 0u;
    // Units of the slices' histograms: places 2 tid and 2 tid + 1 of every ring, requested before any
    // maximum is known, eight slices at a time.
    auto request_units = [&](int s0, uint2 (&hv)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            hv[u] = *reinterpret_cast<const uint2*>(W.hist + (size_t)min(s0 + u, slices - 1) * kPubBins + 2 * tid);
    };
    const bool units = FILTERED ? top_k > 0 : cut;
    uint2 hv[8];
    if (units)
        request_units(0, hv);
    const float M = wave_max_f32(st.max_x);
    if (greedy) {
        const unsigned arg = wave_min_u32(st.max_x == M ? (unsigned)st.argmax : 0xffffffffu);
        if (tid == 0)
            sp.tokens[r] = arg >= 0x7fffffffu ? 0 : max((int)arg - lead, 0);
        return true;
    }
    RowConst rc = row_const(T);
    rc.c_hi = uniform(rc.c_hi);  // (in scalar registers: every vector register counts here)
    rc.c_lo = uniform(rc.c_lo);
    rc.c16 = uniform(rc.c16);
    RowScale rs;
    rs.max_x = M;
    rs.c_hi = rc.c_hi;
    rs.c_lo = rc.c_lo;
    const float kf_row = bin_coord(M, rc.c16), kf_slice = bin_coord(st.max_x, rc.c16);
    const bool empty = st.max_x == -INFINITY;
    // bin b of the slice is bin b + shift of the row
    const int shift = empty ? kBins : (int)fminf(fmaxf(kf_row - kf_slice, 0.f), (float)kBins);
    const int base_slice = ring_base(kf_slice), base_row = ring_base(kf_row);
    auto of_slice = [&](int v, int s) __attribute__((always_inline)) -> int { return __builtin_amdgcn_readlane(v, s); };
    // Row histogram in LDS from the rings: place q of slice s is its bin (base_s - q) mod kPubBins, and
    // the row's bin for that place is (base_row - q) mod kPubBins or that plus kPubBins.
    auto row_histogram = [&](bool as_mass) __attribute__((always_inline)) {
        unsigned long long near[2] = {0ull, 0ull}, far[2] = {0ull, 0ull};
        int rb[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            rb[k] = (base_row - 2 * tid - k) & (kPubBins - 1);
        for (int s0 = 0; s0 < slices; s0 += 8) {
            if (s0 > 0)
                request_units(s0, hv);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (s0 + u >= slices)
                    break;
                const int sh = of_slice(shift, s0 + u), bs = of_slice(base_slice, s0 + u);
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int b = ((bs - 2 * tid - k) & (kPubBins - 1)) + sh;
                    const unsigned v = k ? hv[u].y : hv[u].x;
                    near[k] += b == rb[k] ? v : 0u;
                    far[k] += b == rb[k] + kPubBins ? v : 0u;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            L.row.hist[rb[k]] = (double)near[k] * (as_mass ? bin_unit(rb[k]) : 1.0);
            L.row.hist[rb[k] + kPubBins] = (double)far[k] * (as_mass ? bin_unit(rb[k] + kPubBins) : 1.0);
        }
        __syncthreads();
    };
    static_assert(kPubBins == 2 * kBlock && kBins == 2 * kPubBins, "two places of every ring per thread");

    int lo = kBins, hi = kBins;  // candidate bins, counted down from the maximum's bin; kBins = no cut
    if (cut && !FILTERED) {
        // Estimate of the nucleus cut from the slices' histograms.
        row_histogram(true);
        const BinPick est = block_pick(L.row.hist, 0.0, (double)top_p, true, L.pick);
        // The estimate is good to 3e-5 of the total (a unit is a 32768th of an element at least; a miss is
        // noticed below).  A wider margin takes neighbouring bins in too often: in flat rows, whose bins hold a
        // thousandth of the mass each, three bins did not fit the list (1e-3: 643 rows x 127843 at sigma 1.9,
        // top-p 0.98 752 us, most of them in the whole-row routine).
        const double need_est = (double)top_p * est.total, tol = 1e-4 * est.total;
        lo = hi = __builtin_amdgcn_readfirstlane(est.bin);
        if (need_est - est.above <= tol && lo > 0)
            --lo;
        if (est.above + est.in_bin - need_est <= tol && hi < kBins - 1)
            ++hi;
    }
    // A slice is covered when its emitted bins contain the row's cut bins and everything it summed
    // as above its window is above `lo`.  (A row with a filter is finished from its pairs further down.)
    bool cov = !FILTERED;
    if (cut && !FILTERED)
        cov = st.count >= 0 && st.win_hi >= 0 && (st.win_lo == 0 || st.win_lo + shift <= lo) &&
              (st.win_hi >= kPubBins - 1 || hi <= st.win_hi + shift);
    const unsigned covered = (unsigned)__ballot(cov) & ((1u << slices) - 1u);  // bit s: slice s
    // Bin tests without forming the bin (see the scan kernel): lo == kBins keeps everything,
    // hi == kBins - 1 makes every remaining element a candidate.
    const float t_above = uniform(lo >= kBins ? -INFINITY : kf_row - (float)lo + 1.f);
    const float t_cand = uniform(hi >= kBins - 1 ? -INFINITY : kf_row - (float)hi);

    // ---- mass kept for certain, per 256-element segment in vocabulary order; candidates ----------------
    // The row mass S is put together on the way: exact for every element this kernel sees (the pairs
    // of the covered slices, every logit of the others) and for what the covered slices summed above
    // their windows, estimated from the histograms for the bins past the windows.
    double s_part = 0.0;
    auto take_segment = [&](int sidx, double v) __attribute__((always_inline)) {  // (a wavefront's 64 segments are one slice's)
        if (sidx >= nseg)
            return;
        const int s = __builtin_amdgcn_readfirstlane(sidx / kSegPerSlice);
        const float top = __int_as_float(of_slice(__float_as_int(st.max_x), s));
        v = ((covered >> s) & 1u) && top != -INFINITY ? v * exp2(((double)top - (double)M) * rc.cd) : 0.0;
        seg_mass[sidx] = v;
        s_part += v;
    };
    static_assert(kSegPerSlice == 64, "a wavefront's segments belong to one slice");
    take_segment(tid, seg0);
    if (nseg > kBlock)
        take_segment(tid + kBlock, W.seg[min(tid + kBlock, nseg - 1)]);
    if (cut && tid < slices && ((covered >> tid) & 1u) && !empty)
        // the slice's histogram units refer to 2^(bin_coord(slice max) / 16); the row maximum is 2^(M c16 / 16)
        s_part += st.rest * exp2(((double)kf_slice - (double)M * (double)rc.c16) * 0.0625);
    __syncthreads();
    // One element: kept for certain -> its segment; inside the cut bins -> the candidate list (the
    // lanes of a wavefront take consecutive places reserved with one counter update); else dropped.
    // Called by whole wavefronts (`live` masks lanes that hold nothing).
    float f_part = 0.f;  // exact mass of the elements taken since the last widening
    // (the lane's place among the wavefront's candidates comes from the two lane-count instructions)
    auto append_masked = [&](unsigned long long mask, bool want, unsigned long long pair) __attribute__((always_inline)) {
        if (mask != 0ull) {
            unsigned base = 0u;
            if (lane == 0)
                base = atomicAdd(&L.cand_total, (unsigned)__popcll(mask));
            base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
            if (want) {
                const unsigned pos = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, base));
                if (pos < (unsigned)kCandCap)
                    L.cand[pos] = pair;
            }
        }
    };
    auto take = [&](bool live, float xq, int idx, int s) __attribute__((always_inline)) {
        if (__builtin_amdgcn_ballot_w64(live) == 0ull)
            return;  // nothing in this wavefront's 64 places
        const float t = xq * rc.c16;
        const bool above = live && t >= t_above;
        const bool candq = live && !above && t >= t_cand;
        const float pq = live ? prob(xq, rs) : 0.f;
        f_part += pq;
        if (above)
            atomicAdd(&seg_mass[s * kSegPerSlice + (int)((unsigned)(idx - s * slice_elems) / (unsigned)kSeg)], (double)pq);
        append_masked(__builtin_amdgcn_ballot_w64(candq), candq,
                      (unsigned long long)__float_as_uint(xq) | ((unsigned long long)(unsigned)idx << 32));
    };
    // One wavefront-wide append to the candidate list.
    auto append = [&](bool want, unsigned long long pair) __attribute__((always_inline)) {
        append_masked(__builtin_amdgcn_ballot_w64(want), want, pair);
    };
    // Radix select over the order keys of the first C candidates, taken relative to the largest one
    // (rel = kmax - key, 0 = most probable) so that only the bits in which the candidates differ
    // are resolved: 11 bits per level, usually two levels.  Returns the key of the highest candidate
    // whose upper set (on top of `above0`) reaches `need`, counting candidates (`by_count`) or
    // summing their probabilities; `reached` is what that upper set amounts to, `bad` says that
    // the candidates do not reach `need` at all.
    auto radix_select = [&](int C, bool by_count, double above0, double need, bool& bad, double& reached) -> uint32_t {
        uint32_t kmin = 0xffffffffu, kmax = 0u;
        for (int i = tid; i < C; i += kBlock) {
            const uint32_t key = order_key(__uint_as_float((unsigned)L.cand[i]));
            kmin = min(kmin, key);
            kmax = max(kmax, key);
        }
        kmin = wave_min_u32(kmin);
        kmax = wave_max_u32(kmax);
        __syncthreads();  // an earlier call's readers of kmin / kmax are through
        if (lane == 0) {
            L.kmin[wave] = kmin;
            L.kmax[wave] = kmax;
        }
        if (tid == 0)
            L.members = 0u;
        double* H = L.row.hist;
        for (int b = tid; b < kBins; b += kBlock)
            H[b] = 0.0;
        __syncthreads();
        for (int w = 0; w < kWaves; ++w) {
            kmin = min(kmin, L.kmin[w]);
            kmax = max(kmax, L.kmax[w]);
        }
        const uint32_t span = C > 0 ? kmax - kmin : 0u;
        const int nbits = span ? 32 - __clz((int)span) : 1;
        uint32_t prefix = 0u;
        double abv = above0;
        bad = !(above0 < need);
        const int top_bit = 11 * ((nbits - 1) / 11);
        for (int bit = top_bit; bit >= 0 && !bad; bit -= 11) {
            for (int i = tid; i < C; i += kBlock) {
                const float xc = __uint_as_float((unsigned)L.cand[i]);
                const uint32_t rel = kmax - order_key(xc);
                if ((uint64_t)rel >> (bit + 11) == prefix)
                    atomicAdd(&H[(rel >> bit) & 0x7ffu], by_count ? 1.0 : (double)prob(xc, rs));
            }
            __syncthreads();
            const BinPick pk = block_pick(H, abv, need, false, L.pick);
            // the threshold must fall among the candidates
            if (bit == top_bit && !(above0 + pk.total >= need))
                bad = true;
            prefix = (prefix << 11) | (uint32_t)pk.bin;
            abv = pk.above;
            reached = pk.above + pk.in_bin;
            if (bit == 0 || bad)
                break;
            // The bin usually holds one to three different candidates: up to 64 are told apart directly (every
            // wavefront does it for itself: lane i sums what is not below its own), more take another level.
            unsigned long long* const member = reinterpret_cast<unsigned long long*>(H);
            for (int i = tid; i < C; i += kBlock) {
                const float xc = __uint_as_float((unsigned)L.cand[i]);
                const uint32_t rel = kmax - order_key(xc);
                if (rel >> bit == prefix) {
                    const unsigned at = atomicAdd(&L.members, 1u);
                    if (at < 64u)
                        member[at] = ((unsigned long long)rel << 32) | __float_as_uint(by_count ? 1.f : prob(xc, rs));
                }
            }
            __syncthreads();
            const int members = (int)L.members;
            if (members <= 64) {
                const unsigned long long own = member[max(min(lane, members - 1), 0)];
                const uint32_t rel = (uint32_t)(own >> 32);
                double upper = abv;
                for (int j = 0; j < members; ++j) {
                    const uint32_t rel_j = (uint32_t)__builtin_amdgcn_readlane((int)rel, j);
                    const float p_j = __int_as_float(__builtin_amdgcn_readlane((int)(uint32_t)own, j));
                    upper += rel_j <= rel ? (double)p_j : 0.0;
                }
                // the most probable that reaches `need`; where rounding leaves all of them short, the least
                const uint32_t first = wave_min_u32(upper >= need ? rel : 0xffffffffu);
                prefix = first != 0xffffffffu ? first : wave_max_u32(rel);
                const int at = __ffsll((long long)__ballot(rel == prefix)) - 1;
                reached = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(upper), at),
                                           __builtin_amdgcn_readlane(__double2loint(upper), at));
                __syncthreads();  // (callers and later calls use H again)
                break;
            }
            __syncthreads();
            if (tid == 0)
                L.members = 0u;
            for (int b = tid; b < kBins; b += kBlock)
                H[b] = 0.0;
            __syncthreads();
        }
        return kmax - prefix;
    };
    // pairs written out by the covered slices.  A slice belongs to one wavefront (or to 2, 4, 8 where there are
    // no more than 4, 2, 1 slices), which needs no more of it here than its mass kept for certain, one sum in
    // registers; where in the slice that mass lies is asked of the one slice that the walk ends in.  Two
    // pairs per lane and load, four loads requested ahead (what lies past a slice's count is masked).
    // Candidates are gathered in the wavefront's share of the histogram's place (free until the select) and
    // join the list in one piece: one reservation per step and its round trip took 3 of the 6 us of this
    // phase (64 rows, some 500 candidates each).
    const int wps = slices > 4 ? 1 : slices > 2 ? 2 : slices == 2 ? 4 : 8;  // wavefronts per slice
    constexpr int kStage = kBins / kWaves;
    static_assert(sizeof(L.row.hist[0]) == sizeof(L.cand[0]) && kStage >= 64, "a wavefront's step fits its share");
    unsigned long long* const stage = reinterpret_cast<unsigned long long*>(L.row.hist) + wave * kStage;
    int have = 0;  // (uniform)
    auto flush = [&]() __attribute__((always_inline)) {
        unsigned base = 0u;
        if (lane == 0)
            base = atomicAdd(&L.cand_total, (unsigned)have);
        base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
        for (int i = lane; i < have; i += 64)
            if (base + (unsigned)i < (unsigned)kCandCap)
                L.cand[base + (unsigned)i] = stage[i];
        have = 0;
    };
    for (int round = 0; round < (FILTERED ? 0 : (slices + kWaves - 1) / kWaves); ++round) {
        const int s = round * kWaves + wave / wps, part = wave & (wps - 1);
        double above_mass = 0.0;
        if (s < slices && ((covered >> s) & 1u)) {
            const int cnt = min(of_slice(st.count, s), kEmitCap);
            const ulonglong2* e = reinterpret_cast<const ulonglong2*>(W.emit + (size_t)s * kEmitCap) + 64 * part + lane;
            const int step = 64 * wps, steps = (cnt + 2 * step - 1) / (2 * step);  // (never past the slice's list)
            constexpr int kBatch = 4;
            ulonglong2 now[kBatch], next[kBatch];
            auto request = [&](int i0, ulonglong2 (&v)[kBatch]) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    v[u] = e[(size_t)min(i0 + u, kEmitCap / (2 * step) - 1) * step];
            };
            request(0, now);
            for (int i0 = 0; i0 < steps; i0 += kBatch) {
                request(i0 + kBatch, next);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int first = 2 * ((i0 + u) * step + 64 * part + lane);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const unsigned long long pair = k ? now[u].y : now[u].x;
                        const bool live = first + k < cnt;
                        const float xq = __uint_as_float((unsigned)pair);
                        const float t = xq * rc.c16;
                        const bool above = live && t >= t_above, candq = live && !above && t >= t_cand;
                        const float pq = live ? prob(xq, rs) : 0.f;
                        above_mass += (double)(above ? pq : 0.f);
                        f_part += above ? 0.f : pq;
                        const unsigned long long mask = __builtin_amdgcn_ballot_w64(candq);
                        if (mask != 0ull) {
                            if (have + __popcll(mask) > kStage)
                                flush();
                            if (candq)
                                stage[__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((unsigned)mask, (unsigned)have))] = pair;
                            have += __popcll(mask);
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u)
                    now[u] = next[u];
                s_part += (double)f_part;
                f_part = 0.f;
            }
        }
        if (have > 0)
            flush();
        s_part += above_mass;
        above_mass = wave_scan_f64(above_mass);
        if (lane == 63)
            L.above[round][wave] = above_mass;
    }
    // slices that are not covered: a second look at their logits
    for (int s = 0; s < (FILTERED ? 0 : slices); ++s) {
        if ((covered >> s) & 1u)
            continue;
        const SliceRange g = slice_range(s, slice_elems, V, lead);
        float xv[32];
        SPD_LOAD_SLICE(false, xv, x, g, tid)
        SPD_MASK_SLICE(xv, x, g, tid)
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            const int i = g.e0 + (q >> 2) * kIter + tid * 4 + (q & 3);
            take(i >= lead && i < g.e1, xv[q], i, s);
        }
        s_part += (double)f_part;
        f_part = 0.f;
    }
    uint32_t key_floor = 0u;  // rows with a filter: the lowest key that survives the filters
    if (FILTERED) {
        // ---- min-p and top-k ahead of the nucleus.  Both keep an upper set of the logits, and the scan
        // kernel wrote such a row's slices out from the top, so everything that survives is among the
        // pairs, provided every slice's window reaches as far down as the filters do; otherwise the
        // row goes to the whole-row routine.  Survivors become the candidate list. ----
        bool ok = true;
        // top-k: the k-th largest logit lies in row bins b1 .. b2, by the element-count bounds of the
        // histogram units (an element adds 32768 to 34219 units): the running units reach 32768 k no
        // later than the k-th element's bin and 34219 k no earlier
        int b1 = 0, b2 = 0;
        if (top_k > 0) {
            row_histogram(false);
            const BinPick p1 = block_pick(L.row.hist, 0.0, 32768.0 * (double)top_k, false, L.pick);
            __syncthreads();
            const BinPick p2 = block_pick(L.row.hist, 0.0, 34219.0 * (double)top_k, false, L.pick);
            b1 = p1.bin;
            b2 = p2.bin;
            // fewer than k elements inside the histogram's range: not a case for this path
            ok = ok && p2.total >= 34219.0 * (double)top_k && b2 < kBins - 1;
            __syncthreads();
        }
        // row bin that every slice's window has to reach: the k-th element's, else the last one that
        // can hold p >= min_p (bins are 1/16 octave; two bins of slack for the rounding of p)
        const int reach = top_k > 0 ? b2 : min(kBins - 1, (int)(-__log2f(min_p) * 16.f) + 2);
        const bool reaches = shift >= kBins || (st.count >= 0 && st.win_hi >= 0 && st.win_lo == 0 &&
                                                (st.win_hi >= kPubBins - 1 || st.win_hi + shift >= reach));
        ok = ok && __ballot(reaches) == ~0ull;  // (lanes past the last slice repeat it)
        if (!ok) {
            return false;
        }
        // All pairs of the row, four per thread and slice, those of eight slices requested together; `f(live, pair)` for
        // each.  With top-k they are read twice (the second time from L2): held across the selection between the
        // two they would take 64 registers that it does not have.
        auto for_pairs = [&](auto f) __attribute__((always_inline)) {
            for (int s0 = 0; s0 < slices; s0 += 8) {
                unsigned long long ev[8][4];
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        ev[u][k] = W.emit[(size_t)min(s0 + u, slices - 1) * kEmitCap + tid + k * kBlock];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int s = min(s0 + u, slices - 1);
                    const int cnt = (s0 + u < slices && of_slice(shift, s) < kBins) ? min(of_slice(st.count, s), kEmitCap) : 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        f(tid + k * kBlock < cnt, ev[u][k]);
                }
            }
        };
        uint32_t key_k = 0u;
        if (top_k > 0) {
            // elements above bin b1 are counted, those in b1 .. b2 listed; the k-th largest is found
            // among the listed ones by rank
            const float t_b1 = b1 <= 0 ? INFINITY : kf_row - (float)b1 + 1.f;
            const float t_b2 = kf_row - (float)b2;
            int n_above = 0;
            for_pairs([&](bool live, unsigned long long pair) __attribute__((always_inline)) {
                const float t = __uint_as_float((unsigned)pair) * rc.c16;
                const bool above = live && t >= t_b1;
                n_above += above ? 1 : 0;
                append(live && !above && t >= t_b2, pair);
            });
            double da = (double)n_above, db = 0.0;
            block_sum2_f64(da, db, L.row.scratch);  // (its barriers also complete the list)
            const unsigned listed = L.cand_total;
            const double rank = (double)top_k - da;
            bool bad = listed > (unsigned)kCandCap || rank < 1.0;
            double reached = 0.0;
            if (!bad)
                key_k = radix_select((int)listed, true, 0.0, rank, bad, reached);
            if (bad) {
                return false;
            }
            __syncthreads();
            if (tid == 0)
                L.cand_total = 0u;
            __syncthreads();
        }
        // survivors: at least as large as the k-th largest logit, and p >= min_p
        uint32_t kfl = 0xffffffffu;
        for_pairs([&](bool live, unsigned long long pair) __attribute__((always_inline)) {
            const float xq = __uint_as_float((unsigned)pair);
            const uint32_t key = order_key(xq);
            const float pq = prob(xq, rs);
            const bool keep = live && key >= key_k && pq >= min_p;
            f_part += keep ? pq : 0.f;
            kfl = keep ? min(kfl, key) : kfl;
            append(keep, pair);
        });
        s_part += (double)f_part;
        kfl = wave_min_u32(kfl);
        if (lane == 0)
            L.kmin[wave] = kfl;
        __syncthreads();
        key_floor = 0xffffffffu;
        for (int w = 0; w < kWaves; ++w)
            key_floor = min(key_floor, L.kmin[w]);
        lo = 0;            // no bin is kept wholesale,
        hi = kBins - 1;    // every element is compared with the threshold
    }
    __syncthreads();
    const unsigned cand_total = L.cand_total;
    const int C = (int)min(cand_total, (unsigned)kCandCap);
    // mass kept for certain, slice by slice: the segments that hold some already (what the scan kernel summed
    // above its window, or all of a slice that was read again) and the pairs
    for (int s = wave; s < slices; s += kWaves) {
        double v = wave_scan_f64(seg_mass[s * kSegPerSlice + lane]);
        if (!FILTERED)
            for (int k = 0; k < wps; ++k)
                v += L.above[s / kWaves][s % kWaves * wps + k];
        if (lane == 63)
            L.slice_mass[s] = v;
    }
    s_part = wave_scan_f64(s_part);
    if (lane == 63)
        L.row.scratch[wave] = s_part;
    __syncthreads();
    double above_total = 0.0;
    for (int s = 0; s < slices; ++s)
        above_total += L.slice_mass[s];
    s_part = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        s_part += L.row.scratch[w];
    const double need = (double)top_p * s_part;  // s_part: the row mass S (of what the filters left)

    uint32_t key_tau = key_floor;
    double Z = FILTERED ? s_part : above_total;
    bool bad = cand_total > (unsigned)kCandCap;
    if (cut && !bad) {
        const uint32_t key_cut = radix_select(C, false, above_total, need, bad, Z);
        key_tau = max(key_tau, key_cut);
    }
    if (bad) {
        // candidate overflow or an estimate that missed the cut: redo the row the slow way
        return false;
    }

    // kept candidates join their segments (vocabulary order)
    for (int i = tid; i < C; i += kBlock) {
        const float xc = __uint_as_float((unsigned)L.cand[i]);
        if (order_key(xc) >= key_tau) {
            const int idx = (int)(L.cand[i] >> 32);
            const int s = idx / slice_elems;
            const double pc = (double)prob(xc, rs);
            atomicAdd(&seg_mass[s * kSegPerSlice + (idx - s * slice_elems) / kSeg], pc);
            atomicAdd(&L.slice_mass[s], pc);
        }
    }
    __syncthreads();
    const double target = (double)sp.uniforms[r] * Z;

    // The slice that takes the running mass past the target (rounding may leave the target at the total: then
    // the last one with mass, and its last kept token), and the mass before it.
    int hit = -1;
    double before = 0.0;
    bool take_last = false;
    {
        int last = -1;
        double run = 0.0, before_last = 0.0;
        for (int s = 0; s < slices; ++s) {
            const double m = L.slice_mass[s];
            if (hit < 0 && run + m > target) {
                hit = s;
                before = run;
            }
            if (m > 0.0) {
                last = s;
                before_last = run;
            }
            run += m;
        }
        if (hit < 0) {
            hit = last;
            before = before_last;
            take_last = true;
        }
        hit = __builtin_amdgcn_readfirstlane(hit);
    }
    // Its segments, in vocabulary order: the pairs kept for certain join them.  A wavefront of the scan kernel
    // lists its pairs segment by segment, so a thread's four pairs mostly belong to one segment and go to its
    // sum with one LDS addition per run of equal segments.
    static_assert(kEmitCap == 4 * kBlock, "four pairs per thread");
    if (!FILTERED && hit >= 0 && ((covered >> hit) & 1u)) {
        const int mine = min(max(min(of_slice(st.count, hit), kEmitCap) - 4 * tid, 0), 4);  // of the four places
        if (mine > 0) {
            const ulonglong2* e = reinterpret_cast<const ulonglong2*>(W.emit + (size_t)hit * kEmitCap) + 2 * tid;
            const ulonglong2 lo2 = e[0], hi2 = e[1];
            const unsigned long long ev[4] = {lo2.x, lo2.y, hi2.x, hi2.y};
            double run = 0.0;
            int run_seg = -1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float xq = __uint_as_float((unsigned)ev[k]);
                const int seg = (int)((unsigned)((int)(ev[k] >> 32) - hit * slice_elems) / (unsigned)kSeg);
                if (k < mine && xq * rc.c16 >= t_above) {
                    if (seg != run_seg && run_seg >= 0) {
                        atomicAdd(&seg_mass[hit * kSegPerSlice + run_seg], run);
                        run = 0.0;
                    }
                    run_seg = seg;
                    run += (double)prob(xq, rs);
                }
            }
            if (run_seg >= 0)
                atomicAdd(&seg_mass[hit * kSegPerSlice + run_seg], run);
        }
    }
    lds_barrier();
    if (wave == 0) {
        int seg = -1;
        if (hit >= 0) {
            const double m = seg_mass[hit * kSegPerSlice + lane], inc = before + wave_scan_f64(m);
            const unsigned long long reach = __ballot(inc > target), some = __ballot(m > 0.0);
            take_last = take_last || reach == 0ull;
            const int at = take_last ? (some ? 63 - __clzll((long long)some) : -1) : __ffsll((long long)reach) - 1;
            seg = at < 0 ? -1 : hit * kSegPerSlice + at;
            before = at < 0 ? 0.0 : __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(inc - m), at),
                                                     __builtin_amdgcn_readlane(__double2loint(inc - m), at));
        }
        int token = -1;
        if (seg >= 0) {
            const int s = seg / kSegPerSlice;
            const int base = s * slice_elems + (seg % kSegPerSlice) * kSeg + lane * 4;
            const int end = min(V + lead, (s + 1) * slice_elems);
            float pk[4];
            bool keep[4];
            float s4 = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = base + k;
                pk[k] = 0.f;
                keep[k] = false;
                if (i >= lead && i < end) {
                    const float xi = x[i];
                    const int b = bin_below(kf_row, bin_coord(xi, rc.c16));
                    if (b < lo || (b <= hi && order_key(xi) >= key_tau)) {
                        pk[k] = prob(xi, rs);
                        keep[k] = true;
                        s4 += pk[k];
                    }
                }
            }
            const double inc2 = wave_scan_f64((double)s4);
            double run = before + inc2 - (double)s4;
            int first = 0x7fffffff, lastk = -1;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (keep[k]) {
                    lastk = base + k;
                    run += (double)pk[k];
                    if (run > target && first == 0x7fffffff)
                        first = base + k;
                }
            first = (int)wave_min_u32((unsigned)first);
            lastk = (int)wave_max_u32((unsigned)(lastk + 1)) - 1;
            token = (first != 0x7fffffff && !take_last) ? first : lastk;
        }
        if (lane == 0)
            sp.tokens[r] = token >= 0 ? token - lead : 0;
    }
    return true;
}

// The row-level step is a chain of short dependent phases (a global round trip or an LDS exchange each),
// so what counts is how many there are and how long one takes: scans and reductions stay in registers
// (DPP), a bin is picked by the whole workgroup (8 reads per lane and two barriers instead of 32 reads
// and eleven dependent shuffles in every wavefront), the slices' histograms are requested together with
// their statistics.  Phases of a row of 64 x 128256 (clock stamps, us; before: four pairs of every slice per
// thread, kept mass to its segment, a list reservation per step, every select of two levels): statistics and
// histograms 3.4, pick 1.8, pairs 7.6 -> 4.7, sums 1.9 -> 2.2, select 3.7 -> 3.0, the slice and segment of the
// token 1.0 -> 2.0, walk 1.4.  Whole calls: 64 rows 37.8 -> 36.0 us (33.8 with the narrower margin around the cut, whose
// lists are shorter), 1 row 27.7 -> 25.0, 39 x 167649 39.0 -> 37.3, 300 x 32000 32.9 -> 31.8, 1024 x 128256 204.6 -> 202.3
// (197.5; 194.6 with the logits read past the cache).  Three workgroups share a CU (79 registers, 50 KB of LDS each).
// ANY = false: no row has a filter.  ANY = true (filter arrays are given): every row takes the routine it
// needs in one launch, so that the two kinds run side by side.  Neither instantiation uses scratch memory: the
// filtered routine reads its pairs twice instead of holding them across the selection, and the whole-row
// routine is inlined (a call would have the arguments copied to memory, which every phase then reads).
// (192 rows of 50257 unaligned logits, a third of them each with top-k, min-p and no filter, some greedy:
// whole call 43.8 us, 3 more with the spills; 249 in the whole-row routine.)
template <bool ANY>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) void sampler_finish_kernel(SamplerParams sp, char* ws, int slices, int slice_elems)
{
    __shared__ FinishLds L;
    const long long r = blockIdx.x;
    bool done;
    if (ANY && sp.temperature[r] != 0.f && ((sp.top_k && sp.top_k[r] > 0) || (sp.min_p && sp.min_p[r] > 0.f)))
        done = finish_row<true>(sp, ws, slices, slice_elems, L);
    else
        done = finish_row<false>(sp, ws, slices, slice_elems, L);
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
    // Two workgroups per CU, at most eight slices unless the vocabulary needs more (the row-level
    // step reads every slice's histogram), and no slice shorter than 4096 logits.
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
    // Rows that do not all start on a 16-byte boundary are cut in positions counted from the boundary
    // before each (up to three more than the vocabulary).
    const bool aligned = (p.stride % 4 == 0) && ((uintptr_t)p.logits % 16 == 0);
    const long long span = aligned ? p.vocab : p.vocab + 3;
    // Short rows that are not aligned take the whole-row kernel, one launch whose passes all hit the L2.  The
    // two sides at 64 rows: 2001 logits 17.7 us against 19.2 in the sliced kernels, 4001 20.8 / 19.8, 5001
    // 22.7 / 19.2; without a cut 4001 9.5 / 10.1, 5001 10.7 / 9.9; with filters 5001 31.9 / 33.0, 7001 38.5 / 33.0;
    // the lines lie within 1000 logits of these from 1 to 2048 rows, except near 768.  (Greedy rows alone
    // would cross at 11000, 4.6 / 5.9 us at 5001: they are not known here.)
    const bool filters = p.top_k || p.min_p;
    const long long least = aligned ? 4 : filters ? 6144 : 4096;
    if (slices == 0 || span > (long long)slices * kSliceMax || p.vocab < least) {
        hipLaunchKernelGGL(sample_rows_kernel, dim3((unsigned)p.rows), dim3(kBlock), 0, s, p);
        return hipGetLastError();
    }
    int slice_elems = (int)((span + slices - 1) / slices);
    slice_elems = (slice_elems + 3) / 4 * 4;
    // Logits that the last-level cache (256 MB) cannot hold are read past it: 1024 x 128256 (525 MB) 207 -> 202 us;
    // 64 x 128256 (33 MB, where the LM head has just left them) would lose, 38.9 / 39.9.
    const bool stream = 4.0 * (double)p.rows * (double)p.vocab >= 256e6;
    hipLaunchKernelGGL(stream ? sampler_scan_kernel<true> : sampler_scan_kernel<false>, dim3((unsigned)(p.rows * slices)), dim3(kBlock), 0, s, p, (char*)ws, slices,
                       slice_elems);
    if (filters)
        hipLaunchKernelGGL(sampler_finish_kernel<true>, dim3((unsigned)p.rows), dim3(kBlock), 0, s, p, (char*)ws,
                           slices, slice_elems);
    else
        hipLaunchKernelGGL(sampler_finish_kernel<false>, dim3((unsigned)p.rows), dim3(kBlock), 0, s, p, (char*)ws,
                           slices, slice_elems);
    return hipGetLastError();
}

}  // namespace spd
