// Exact SURE threshold by histogram search.
//
// For coefficients b_1..b_N of one component the risk estimate of soft
// thresholding at unit noise is SURE(t) = N - 2 #{|b| <= t} + sum min(b^2, t^2).
// Between consecutive candidates t in {0} U {|b_k|} it increases with t, so the
// minimum is attained on the candidate set.
//
// The magnitude |b| is keyed by its IEEE bit pattern (monotone for
// non-negative numbers); exact zeros are only counted.  A bin of keys [lo, hi)
// that holds c of the values, with C values below it whose squares sum to S, has
//   N - 2 (C + c) + S + (N - C) lo^2                    (L)
// as a lower bound of SURE over the candidates in it, and with s the sum of
// squares inside, t the largest number below hi,
//   N - 2 (C + c) + S + s + (N - C - c) t^2             (U)
// as an upper bound of the minimum.  A bin whose L exceeds a known U is out.
//
// 1. k_sure_hist (components of more than kSureDirect values): counts per bin
//    of each chunk, one LDS atomic per value, into a row of its own.
// 2. k_sure_gather: every block adds its component's rows, finds the range of
//    the surviving bins, and copies its chunk's values in that range into its
//    segment of a list, with the sum of squares of those below; tied values go
//    there as pairs of value and count.
//    Beyond kSureLarge values k_sure_rows adds the rows up first, and rounds of
//    k_sure_refine and k_sure_narrow shorten the list before step 3.
// 3. k_sure_finish, one block per component: histograms of counts and sums of
//    squares over the list, each over the range that survived, until the
//    surviving bins are small; their values, grouped by bin in LDS, are then
//    evaluated one by one.  Too many survivors all over a range are searched in
//    windows of it.  Smaller components do step 1 here, over the coefficients
//    themselves.
//
// The first histogram has 512 bins per octave of [1/16, 8), where thresholds
// of unit-noise coefficients lie (lower for components of smaller values): 16 per octave (one key range for all numbers)
// put most values of a block into some fifty bins, whose LDS atomics queued,
// and left most of the values to a second full histogram.  Its sums are not
// needed: the squares of a bin lie between those of its edges, and a bin is
// compared with the best one through the bins between the two.
//
// Bound by latency and LDS atomics: the three passes over the 21 MB of 349 x 1905
// and 8 components take 10, 23 and 43 us, against 145 us for six passes with a
// select in the last block of each; ten components of 145 x 217, one launch,
// 37 us against 594; four FP64 ones of 64 x 64 25 us against 158.
#include <type_traits>

#include "hyres_internal.hpp"

namespace hyres {

constexpr int kSureThreads = 1024;
constexpr int kSureWaves = kSureThreads / 64;
constexpr int kBinsPer = kSureBins / kSureThreads;    // bins per thread in the selects
constexpr int kSureLoads = 16;       // values a thread reads at once
constexpr int kZeroSlot = kSureBins - 1;              // first histogram: exact zeros
constexpr int kSureLight = 64;      // largest bin evaluated without narrowing the range first
constexpr int kSureHeavy = 256;     // a larger bin is searched as a range of its own
constexpr int kSureHeavies = 16;    // ... up to this many of them; more, or more values than fit in LDS: windows
constexpr int kSureWindows = 16;
constexpr int kSureStack = 256;     // ranges waiting
// Values the finish reads in all, in passes over its list, before it gives the
// smallest risk seen (1.5 ms of one block).  Only a risk that is flat over much of its
// range gets there: of Rayleigh-distributed magnitudes, whose expected risk is the
// same everywhere, a million are finished in 1.0-1.6 ms (bin by bin 1-55).
constexpr int64_t kSureVisits = (int64_t)1 << 23;

// Keys, and the bins of the first histogram: 512 per octave in the seven octaves
// from `fine` on, kSureOuter bits wide below and above.  Word: the part of the key the
// bins are formed from (its high word for FP64).
template <typename T> struct KeyTraits;
template <> struct KeyTraits<float> {
    typedef uint32_t K;
    static constexpr int kCap = 16384;       // values evaluated at once (LDS)
    static constexpr int kWordShift = 0;
    static constexpr int kOctave = 23;       // bits of an octave in a word
    static constexpr uint32_t kFine = 0x3D800000u;       // 1/16
    __device__ static K key(float v) { return __float_as_uint(v) & 0x7fffffffu; }
    __device__ static double val(uint64_t k) { return (double)__uint_as_float((uint32_t)k); }
};
template <> struct KeyTraits<double> {
    typedef unsigned long long K;
    static constexpr int kCap = 8192;
    static constexpr int kWordShift = 32;
    static constexpr int kOctave = 20;
    static constexpr uint32_t kFine = 0x3FB00000u;
    __device__ static K key(double v) {
        return (unsigned long long)__double_as_longlong(v) & 0x7fffffffffffffffull;
    }
    __device__ static double val(uint64_t k) { return __longlong_as_double((long long)k); }
};
constexpr int kSureOuter = 22;               // bits of an outer bin
constexpr int kSureOctaves = 7;              // ... of 512 bins
// Words of those octaves, and the first bin of them
template <typename T> constexpr uint32_t kFineSpan = (uint32_t)kSureOctaves << KeyTraits<T>::kOctave;
__device__ __forceinline__ int fine_bin(uint32_t fine) { return (int)((fine + (1u << kSureOuter) - 1) >> kSureOuter); }
template <typename T>
__device__ __forceinline__ int first_bin(typename KeyTraits<T>::K k, uint32_t fine) {
    typedef KeyTraits<T> KT;
    const uint32_t w = (uint32_t)((uint64_t)k >> KT::kWordShift);
    if (w < fine) return (int)(w >> kSureOuter);
    const int low = fine_bin(fine);
    if (w - fine < kFineSpan<T>) return low + (int)((w - fine) >> (KT::kOctave - 9));
    return low + kSureOctaves * 512 + (int)((w - fine - kFineSpan<T>) >> kSureOuter);
}
// Smallest key of bin b (the end of the keys beyond the last bin).
template <typename T>
__device__ __forceinline__ uint64_t first_edge(int b, uint32_t fine) {
    typedef KeyTraits<T> KT;
    const int low = fine_bin(fine), high = low + kSureOctaves * 512;
    uint64_t w;
    if (b < low) w = (uint64_t)b << kSureOuter;
    else if (b < high) w = fine + ((uint64_t)(b - low) << (KT::kOctave - 9));
    else w = (uint64_t)fine + kFineSpan<T> + ((uint64_t)(b - high) << kSureOuter);
    if (w > 0x80000000ull) w = 0x80000000ull;
    return w << KT::kWordShift;
}

// Smallest shift that leaves at most kSureBins bins of a span > 0.
__device__ __forceinline__ int shift_for(uint64_t span) {
    static_assert(kSureBins == 1 << 12, "12 bits of bins");
    const int len = span > 1 ? 64 - __clzll((long long)(span - 1)) : 0;
    return len > 12 ? len - 12 : 0;
}

__device__ __forceinline__ int64_t sure_count(const CubeDesc& d) {
    return d.scope == HYRES_SCOPE_DETAIL ? d.ll_off : d.nc;
}

// ---- wave primitives (whole wave active) ----
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
// Inclusive prefix sums over the 64 lanes: rows by DPP row shifts, then the
// totals of the rows before (fixed order).
__device__ __forceinline__ uint32_t wave_incl_u32(uint32_t v) {
    v += dpp_u32<0x111>(v);
    v += dpp_u32<0x112>(v);
    v += dpp_u32<0x114>(v);
    v += dpp_u32<0x118>(v);
    const uint32_t t0 = readlane_u32(v, 15), t1 = readlane_u32(v, 31), t2 = readlane_u32(v, 47);
    const int row = (threadIdx.x & 63) >> 4;
    uint32_t off = row >= 1 ? t0 : 0u;
    off += row >= 2 ? t1 : 0u;
    off += row >= 3 ? t2 : 0u;
    return v + off;
}
__device__ __forceinline__ double wave_incl_f64(double v) {
    v += dpp_shift_f64<0x111>(v);
    v += dpp_shift_f64<0x112>(v);
    v += dpp_shift_f64<0x114>(v);
    v += dpp_shift_f64<0x118>(v);
    const double t0 = readlane_f64(v, 15), t1 = readlane_f64(v, 31), t2 = readlane_f64(v, 47);
    const int row = (threadIdx.x & 63) >> 4;
    double off = row >= 1 ? t0 : 0.0;
    off = row >= 2 ? off + t1 : off;
    off = row >= 3 ? off + t2 : off;
    return v + off;
}
// (value, t) pairs: smaller value, then smaller t, over the wave (every lane gets it)
__device__ __forceinline__ void wave_argmin(double& b, double& t) {
#define HYRES_AM(CTRL)                                                 \
    {                                                                  \
        const double ob = dpp_f64<CTRL>(b), ot = dpp_f64<CTRL>(t);    \
        if (ob < b || (ob == b && ot < t)) { b = ob; t = ot; }         \
    }
    HYRES_AM(0xB1) HYRES_AM(0x4E) HYRES_AM(0x141) HYRES_AM(0x140)
#undef HYRES_AM
    double bb = readlane_f64(b, 0), tt = readlane_f64(t, 0);
    for (int r = 16; r < 64; r += 16) {
        const double ob = readlane_f64(b, r), ot = readlane_f64(t, r);
        if (ob < bb || (ob == bb && ot < tt)) { bb = ob; tt = ot; }
    }
    b = bb;
    t = tt;
}
template <bool MAX>
__device__ __forceinline__ int wave_minmax_i32(int v) {
#define HYRES_MM(CTRL)                                                         \
    {                                                                          \
        const int o = (int)dpp_u32<CTRL>((uint32_t)v);                          \
        v = MAX ? (o > v ? o : v) : (o < v ? o : v);                           \
    }
    HYRES_MM(0xB1) HYRES_MM(0x4E) HYRES_MM(0x141) HYRES_MM(0x140)
#undef HYRES_MM
    int r = __builtin_amdgcn_readlane(v, 0);
    for (int l = 16; l < 64; l += 16) {
        const int o = __builtin_amdgcn_readlane(v, l);
        r = MAX ? (o > r ? o : r) : (o < r ? o : r);
    }
    return r;
}


// Small per-block state.
struct SureShared {
    uint32_t wc[kSureWaves], wn[kSureWaves], wm[kSureWaves];
    double ws[kSureWaves], wt[kSureWaves], bs[kSureWaves], bt[kSureWaves];
    int wf[kSureWaves], wl[kSureWaves], wx[kSureWaves];
    uint32_t zeros, count, pairs;
    int tied;
    double ref[4];                 // first select: the reference bin
    uint64_t c0;
    int first, last;
};

// Combining one value per wave (in LDS, kSureWaves = 16 of them) in a DPP row:
// every wave does it for itself, one LDS read and four steps.
static_assert(kSureWaves == 16, "one DPP row");
// sum of the waves before this one; the sum of all in *total
__device__ __forceinline__ uint32_t waves_before(const uint32_t* w, int wave, uint32_t* total) {
    uint32_t v = w[threadIdx.x & 15];
    v += dpp_u32<0x111>(v);
    v += dpp_u32<0x112>(v);
    v += dpp_u32<0x114>(v);
    v += dpp_u32<0x118>(v);
    *total = readlane_u32(v, 15);
    return wave ? readlane_u32(v, wave - 1) : 0u;
}
__device__ __forceinline__ double waves_before(const double* w, int wave, double* total) {
    double v = w[threadIdx.x & 15];
    v += dpp_shift_f64<0x111>(v);
    v += dpp_shift_f64<0x112>(v);
    v += dpp_shift_f64<0x114>(v);
    v += dpp_shift_f64<0x118>(v);
    *total = readlane_f64(v, 15);
    return wave ? readlane_f64(v, wave - 1) : 0.0;
}
template <bool MAX>
__device__ __forceinline__ int waves_minmax(const int* w) {
    return wave_minmax_i32<MAX>(w[threadIdx.x & 15]);
}

// First histogram of values e0..e1-1 into lc (kSureBins counts, zeroed by the
// caller).  Each thread keeps its zeros; returns them.
template <typename T, int U>
__device__ __forceinline__ uint32_t first_histogram_u(const HYRES_GLOBAL T* cf, int64_t e0, int64_t e1, uint32_t fine, uint32_t* lc) {
    typedef KeyTraits<T> KT;
    uint32_t nz = 0;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += U * kSureThreads) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = e + (int64_t)u * kSureThreads;
            v[u] = cf[i < e1 ? i : e1 - 1];          // unconditional: see k_sure_gather
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const auto k = KT::key(e + (int64_t)u * kSureThreads < e1 ? v[u] : (T)0);
            if (k != 0) atomicAdd(&lc[first_bin<T>(k, fine)], 1u);
            else if (e + (int64_t)u * kSureThreads < e1) ++nz;
        }
    }
    return nz;
}
// Up to four values a thread are not read sixteen at a time, whose clamped loads and
// zeros take 1.3 us more (27.5 and 28.9 us for four components of 4096; eight at a
// time up to 8192 would save 0.9 there, and cost FP64 searches of any size 0.3).
template <typename T>
__device__ __forceinline__ uint32_t first_histogram(const HYRES_GLOBAL T* cf, int64_t e0, int64_t e1, uint32_t fine, uint32_t* lc) {
    return e1 - e0 <= 4 * kSureThreads ? first_histogram_u<T, 4>(cf, e0, e1, fine, lc)
                                       : first_histogram_u<T, kSureLoads>(cf, e0, e1, fine, lc);
}

// Whether a thread's bins among first..last show tied values: a bin of more than 64
// with an empty one beside it, which a continuous distribution does not leave, or
// alone in the range.
__device__ __forceinline__ bool bins_tied(const uint32_t (&c)[kBinsPer], int first, int last) {
    bool heavy = false, gap = first == last;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j) {
        const int b = kBinsPer * (int)threadIdx.x + j;
        const bool in = b >= first && b <= last;
        heavy |= in && c[j] > 64;
        gap |= in && c[j] == 0;
    }
    return heavy && gap;
}

// Select on the first histogram: c[j] holds bin 4 tid + j (the zero slot's
// count in `zeros`).  Returns the first and last surviving bin (-1: none) and the
// number of values below the first.  Sums of squares are known to the edges of
// the bins only: relative to a reference bin J with upper bound U, L - U needs
// the sum over the bins between, bounded by their edges.
// TIES: sh.tied (cleared before) tells whether a bin shows tied values.
template <typename T, bool TIES>
__device__ __forceinline__ void first_select(const uint32_t (&c)[kBinsPer], uint32_t zeros, double N, uint32_t fine,
                                             SureShared& sh, int* first, int* last, uint64_t* c0) {
    typedef KeyTraits<T> KT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double a[kBinsPer], b[kBinsPer];
    uint32_t tc = 0;
    double tl = 0.0, th = 0.0;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j) {
        const int bin = kBinsPer * tid + j;
        const double lo = KT::val(first_edge<T>(bin, fine)), hi = KT::val(first_edge<T>(bin + 1, fine) - 1);
        a[j] = lo * lo;
        b[j] = hi * hi;
        if (c[j]) {
            tc += c[j];
            tl = fma((double)c[j], a[j], tl);
            th = fma((double)c[j], b[j], th);
        }
    }
    const uint32_t ic = wave_incl_u32(tc);
    const double il = wave_incl_f64(tl), ih = wave_incl_f64(th);
    const double pl = __shfl_up(il, 1, 64), ph = __shfl_up(ih, 1, 64);
    if (lane == 63) {
        sh.wc[wave] = ic;
        sh.ws[wave] = il;
        sh.wt[wave] = ih;
    }
    __syncthreads();
    uint32_t all;
    double allf;
    const uint32_t oc = waves_before(sh.wc, wave, &all);
    const double ol = waves_before(sh.ws, wave, &allf), oh = waves_before(sh.wt, wave, &allf);
    // values below this thread's bins, and the bounds of their sum of squares
    const double C0 = (double)zeros + (double)(oc + ic - tc);
    const double L0 = lane ? ol + pl : ol, H0 = lane ? oh + ph : oh;
    double best = __builtin_inf(), bj = 0.0;
    {
        double C = C0, Sl = L0, Sh = H0;
#pragma unroll
        for (int j = 0; j < kBinsPer; ++j) {
            if (!c[j]) continue;
            C += c[j];
            Sl = fma((double)c[j], a[j], Sl);
            Sh = fma((double)c[j], b[j], Sh);
            const double e = N - 2.0 * C + 0.5 * (Sl + Sh) + (N - C) * b[j];
            if (e < best) {
                best = e;
                bj = (double)(kBinsPer * tid + j);
            }
        }
    }
    wave_argmin(best, bj);
    if (lane == 0) {
        sh.bs[wave] = best;
        sh.bt[wave] = bj;
    }
    __syncthreads();
    best = sh.bs[lane & 15];
    bj = sh.bt[lane & 15];
    wave_argmin(best, bj);
    const int J = (int)bj;
    if (tid == J / kBinsPer) {
        double C = C0, Sl = L0, Sh = H0, bb = 0.0;
#pragma unroll
        for (int j = 0; j < kBinsPer; ++j)
            if (kBinsPer * tid + j <= J && c[j]) {
                C += c[j];
                Sl = fma((double)c[j], a[j], Sl);
                Sh = fma((double)c[j], b[j], Sh);
                bb = b[j];
            }
        sh.ref[0] = C;
        sh.ref[1] = Sl;
        sh.ref[2] = Sh;
        sh.ref[3] = bb;
    }
    __syncthreads();
    const double CJ = sh.ref[0], SlJ = sh.ref[1], ShJ = sh.ref[2], rise = (N - CJ) * sh.ref[3];
    const bool have = best < __builtin_inf();
    const double tol = 1e-10 * (N + ShJ + rise);
    int f = 0x7fffffff, l = -1;
    double cf = 0.0;
    {
        double C = C0, Sl = L0, Sh = H0;
#pragma unroll
        for (int j = 0; j < kBinsPer; ++j) {
            const int bin = kBinsPer * tid + j;
            if (!c[j]) continue;
            const double cc = (double)c[j], low = (N - C) * a[j];
            const double between = bin > J ? Sl - SlJ : Sh - ShJ;
            const double over = -2.0 * (C + cc - CJ) + between + low - rise;        // L - U at the reference
            const double over0 = -2.0 * (C + cc - (double)zeros) + Sl + low;        // L - SURE(0)
            if (have && over <= tol && over0 <= tol) {     // NaN: not a candidate
                if (bin < f) {
                    f = bin;
                    cf = C;
                }
                l = bin;
            }
            C += cc;
            Sl = fma(cc, a[j], Sl);
            Sh = fma(cc, b[j], Sh);
        }
    }
    const int wf = wave_minmax_i32<false>(f), wl = wave_minmax_i32<true>(l);
    if (lane == 0) {
        sh.wf[wave] = wf;
        sh.wl[wave] = wl;
    }
    __syncthreads();
    const int ff = waves_minmax<false>(sh.wf), ll = waves_minmax<true>(sh.wl);
    if (l >= 0 && f == ff) sh.c0 = (uint64_t)cf;
    if (TIES && bins_tied(c, ff, ll)) sh.tied = 1;
    __syncthreads();
    *first = ll >= 0 ? ff : -1;
    *last = ll;
    *c0 = sh.c0;
}

// Keys of the bins first..last, zeros left out.
template <typename T>
__device__ __forceinline__ void first_range(int first, int last, uint32_t fine, uint64_t* klo, uint64_t* khi) {
    const uint64_t k = first_edge<T>(first, fine);
    *klo = k ? k : 1;
    *khi = first_edge<T>(last + 1, fine);
}

// First word of the octaves of 512 bins for a component of N > kSureDirect values, from
// 64 of them, the same for every wave: 1/16, but where the largest of the 64 is below
// that (and not zero), 1/32 to 1/64 of it.  The risk of values far below the noise
// falls up to the largest of them, and with 1/16 a million FP64 ones of standard
// deviation 0.001 share a few bins: the search took 0.6 ms, of equally spaced values
// 2.1, most of it the one finishing block (0.06, 0.07).  Values far above it leave the
// first few: nothing to gain.
template <typename T>
__device__ __forceinline__ uint32_t sure_fine(T v) {
    typedef KeyTraits<T> KT;
    const uint32_t w = (uint32_t)wave_minmax_i32<true>((int)(uint32_t)((uint64_t)KT::key(v) >> KT::kWordShift));
    const uint32_t octave = w >> KT::kOctave << KT::kOctave, below = 5u << KT::kOctave;
    return w >= KT::kFine || w == 0 ? KT::kFine : octave > below ? octave - below : 0u;
}

template <typename T>
__global__ __launch_bounds__(kSureThreads) void k_sure_hist(const CubeDesc* __restrict__ descs,
                                                            const int* __restrict__ items, int ncubes) {
    __shared__ __align__(16) uint32_t lc[kSureBins];
    const int c = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[c];
    const int nch = d.snch, local = blockIdx.x - items[c], comp = local / nch, chunk = local - comp * nch;
    const int tid = threadIdx.x;
    const int64_t N = sure_count(d), e0 = (int64_t)chunk * d.schunk, e1 = min(e0 + d.schunk, N);
    const HYRES_GLOBAL T* cf = gmem(static_cast<const T*>(d.coef)) + (int64_t)comp * d.ncs;
    static_assert(kSureDirect >= 64 * 64, "the sample's last is below N");
    const T sample = cf[(tid & 63) * (N / 64) + (29 * tid & 63)];
    for (int b = tid; b < kSureBins; b += kSureThreads) lc[b] = 0;
    __syncthreads();
    const uint32_t fine = sure_fine<T>(sample);
    if (chunk == 0 && tid == 0) d.ssel[comp * (d.srounds + 1)].fine = fine;
    const uint32_t nz = first_histogram<T>(cf, e0, e1, fine, lc);
    if (nz) atomicAdd(&lc[kZeroSlot], nz);
    __syncthreads();
    HYRES_GLOBAL uint32_t* row = gmem(d.shist) + comp * d.shcs;
    if (d.schunk <= kSureRow16) {             // counts of a chunk fit 16 bits: two per word
        row += (int64_t)chunk * (kSureBins / 2);
        for (int b = tid; b < kSureBins / 2; b += kSureThreads) row[b] = lc[2 * b] | lc[2 * b + 1] << 16;
    } else {
        row += (int64_t)chunk * kSureBins;
        for (int b = tid; b < kSureBins; b += kSureThreads) row[b] = lc[b];
    }
}

// Appends the values of [klo, khi) among a wave's v (zeros are in no range) to a
// list of `cap` values; *count counts those beyond it too.
template <typename T, int U, typename C>
__device__ __forceinline__ void keep_values(const T (&v)[U], const bool (&in)[U], HYRES_GLOBAL T* list, uint32_t cap,
                                            C* count) {
    const int lane = threadIdx.x & 63;
    uint32_t n = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) n += (uint32_t)__popcll(__ballot(in[u]));
    if (!n) return;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(count, n);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const unsigned long long m = __ballot(in[u]);
        const uint32_t pos = at + (uint32_t)__popcll(m & ((1ull << lane) - 1));
        if (in[u] && pos < cap) list[pos] = v[u];
        at += (uint32_t)__popcll(m);
    }
}
template <typename T, int U, typename C>
__device__ __forceinline__ void keep_range(const T (&v)[U], uint64_t klo, uint64_t khi, HYRES_GLOBAL T* list, uint32_t cap,
                                           C* count) {
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t k = KeyTraits<T>::key(v[u]);
        in[u] = k >= klo && k < khi;
    }
    keep_values<T, U>(v, in, list, cap, count);
}

// ---- components of tied values (integers, a quantised image) ----
// A bin then holds one value many times over, and a list of them all is most of the
// component: one block took 2 ms for a million integers, 32 for 2^24 (0.3 and 0.46 in
// passes over all of them by all blocks).  A block keeps one value per bin instead,
// the first it meets, and counts those equal to it; at its end they go to the list as
// pairs of value and count, from the end of the list's space downwards: a million
// integers 0.1 ms, 2^24 0.2.
template <typename T>
struct SureTies {
    typename KeyTraits<T>::K key[kSureBins];
    uint32_t n[kSureBins];
};
template <typename T>
__device__ __forceinline__ void clear_ties(SureTies<T>& t) {      // a barrier follows
    for (int b = threadIdx.x; b < kSureBins; b += kSureThreads) {
        t.key[b] = 0;
        t.n[b] = 0;
    }
}
// The values p[0..m) of [klo, khi) kept so; returns the squares of those below.
template <typename T, typename Bin, typename C>
__device__ __forceinline__ double fold_ties(const HYRES_GLOBAL T* p, int64_t m, uint64_t klo, uint64_t khi, SureTies<T>& t,
                                            Bin bin, HYRES_GLOBAL T* list, uint32_t cap, C* count) {
    typedef typename KeyTraits<T>::K K;
    const int lane = threadIdx.x & 63;
    double below = 0.0;
    for (int64_t e = threadIdx.x - lane; e < m; e += 4 * kSureThreads) {     // whole waves
        T v[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = e + lane + (int64_t)u * kSureThreads;
            v[u] = p[i < m ? i : m - 1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (e + lane + (int64_t)u * kSureThreads >= m) v[u] = (T)0;
            const K k = KeyTraits<T>::key(v[u]);
            in[u] = (uint64_t)k >= klo && (uint64_t)k < khi;
            if ((uint64_t)k < klo) below = fma((double)v[u], (double)v[u], below);
            if (in[u]) {
                const int b = bin(k);
                K r = t.key[b];
                if (r == 0) {
                    const K old = atomicCAS(&t.key[b], (K)0, k);
                    r = old ? old : k;
                }
                if (r == k) {
                    atomicAdd(&t.n[b], 1u);
                    in[u] = false;
                }
            }
        }
        keep_values<T, 4>(v, in, list, cap, count);
    }
    return below;
}
// (after a barrier)  `end` is the end of a list's space of `cap` values.
template <typename T, typename C>
__device__ __forceinline__ void keep_ties(const SureTies<T>& t, HYRES_GLOBAL T* end, int64_t cap, C* pairs) {
    for (int b = threadIdx.x; b < kSureBins; b += kSureThreads)
        if (t.n[b]) {
            const int64_t at = 2 * (int64_t)(atomicAdd(pairs, 1u) + 1u);
            if (at <= cap) {
                end[-at] = (T)KeyTraits<T>::val(t.key[b]);
                end[1 - at] = (T)t.n[b];          // below 2^24: exact
            }
        }
}

// Large components (d.srounds > 0): the chunks' count rows added into one, which the
// gather reads, and the rows and list lengths of the refining rounds cleared.
// kSureSplit blocks per component, each 64 bins: 16 threads of four bins
// by 16 shares of the rows (256 rows in 5 us; one bin and all rows a thread took 30).
template <typename T>
__global__ __launch_bounds__(256) void k_sure_rows(const CubeDesc* __restrict__ descs, const int* __restrict__ items,
                                                   int ncubes) {
    __shared__ uint32_t part[16][64];
    const int cu = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[cu];
    const int local = blockIdx.x - items[cu], comp = local / kSureSplit, b0 = (local - comp * kSureSplit) * 64;
    static_assert(kSureBins == kSureSplit * 64, "64 bins a block");
    const int tid = threadIdx.x, bin = b0 + 4 * (tid & 15), share = tid >> 4;
    HYRES_GLOBAL uint32_t* rows = gmem(d.shist) + comp * d.shcs;
    uint32_t c[4] = {0, 0, 0, 0};
    if (d.schunk <= kSureRow16) {
        const HYRES_GLOBAL uint64_t* r = (const HYRES_GLOBAL uint64_t*)rows + bin / 4;
#pragma unroll 16
        for (int k = share; k < d.snch; k += 16) {
            const uint64_t w = r[(int64_t)k * (kSureBins / 4)];
            c[0] += (uint32_t)w & 0xffffu;
            c[1] += (uint32_t)w >> 16;
            c[2] += (uint32_t)(w >> 32) & 0xffffu;
            c[3] += (uint32_t)(w >> 48);
        }
    } else {
        typedef uint32_t U4 __attribute__((ext_vector_type(4)));
        const HYRES_GLOBAL U4* r = (const HYRES_GLOBAL U4*)rows + bin / 4;
#pragma unroll 16
        for (int k = share; k < d.snch; k += 16) {
            const U4 w = r[(int64_t)k * (kSureBins / 4)];
            c[0] += w[0];
            c[1] += w[1];
            c[2] += w[2];
            c[3] += w[3];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) part[share][4 * (tid & 15) + j] = c[j];
    __syncthreads();
    HYRES_GLOBAL uint32_t* out = rows + (int64_t)d.snch * kSureBins;
    if (tid < 64) {
        uint32_t t = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += part[k][tid];
        out[b0 + tid] = t;
    }
    for (int k = tid; k < 3 * kSureRefine * 64; k += 256) out[(1 + k / 64) * kSureBins + b0 + k % 64] = 0u;
    if (b0 == 0 && tid <= d.srounds) {
        d.ssel[comp * (d.srounds + 1) + tid].count = 0u;
        d.ssel[comp * (d.srounds + 1) + tid].pairs = 0u;
    }
}

template <typename T>
__global__ __launch_bounds__(kSureThreads) void k_sure_gather(const CubeDesc* __restrict__ descs,
                                                              const int* __restrict__ items, int ncubes) {
    typedef KeyTraits<T> KT;
    __shared__ SureShared sh;
    __shared__ SureTies<T> ties;
    const int cu = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[cu];
    const int nch = d.snch, local = blockIdx.x - items[cu], comp = local / nch, chunk = local - comp * nch;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t N = sure_count(d);
    const int64_t e0 = (int64_t)chunk * d.schunk, e1 = min(e0 + d.schunk, N);
    const HYRES_GLOBAL T* cf = gmem(static_cast<const T*>(d.coef)) + (int64_t)comp * d.ncs;
    constexpr int U = kSureLoads;
    T v[U];
    // every load unconditional (clamped): loads under a condition wait for one another
    auto fetch = [&](int64_t e) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = e + lane + (int64_t)u * kSureThreads;
            v[u] = cf[i < e1 ? i : N - 1];
        }
    };
    SureSel* s = d.ssel + comp * (d.srounds + 1);
    const uint32_t fine = s->fine;
    uint32_t c[kBinsPer] = {0, 0, 0, 0};
    static_assert(kBinsPer == 4, "rows are read four bins at a time");
    const HYRES_GLOBAL uint32_t* rows = gmem(d.shist) + comp * d.shcs;
    if (d.srounds) {
        const HYRES_GLOBAL uint32_t* r = rows + (int64_t)nch * kSureBins + kBinsPer * tid;
#pragma unroll
        for (int j = 0; j < kBinsPer; ++j) c[j] = r[j];
    } else if (d.schunk <= kSureRow16) {
        const HYRES_GLOBAL uint64_t* r = (const HYRES_GLOBAL uint64_t*)rows + tid;
        for (int k = 0; k < nch; k += 16) {
            uint64_t x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) x[q] = r[(int64_t)min(k + q, nch - 1) * kSureThreads];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const uint64_t w = k + q < nch ? x[q] : 0;
                c[0] += (uint32_t)w & 0xffffu;
                c[1] += (uint32_t)w >> 16;
                c[2] += (uint32_t)(w >> 32) & 0xffffu;
                c[3] += (uint32_t)(w >> 48);
            }
        }
    } else {
#pragma unroll 4
        for (int k = 0; k < nch; ++k)
#pragma unroll
            for (int j = 0; j < kBinsPer; ++j) c[j] += rows[(int64_t)k * kSureBins + kBinsPer * tid + j];
    }
    if (tid == kSureThreads - 1) {
        sh.zeros = c[kBinsPer - 1];
        c[kBinsPer - 1] = 0;
        sh.count = 0;
        sh.pairs = 0;
        sh.tied = 0;
    }
    __syncthreads();
    const uint32_t zeros = sh.zeros;
    int first, last;
    uint64_t c0;
    fetch(e0 + tid - lane);                  // under the selection
    first_select<T, true>(c, zeros, (double)N, fine, sh, &first, &last, &c0);
    uint64_t klo = 1, khi = 1;
    if (first >= 0) first_range<T>(first, last, fine, &klo, &khi);
    if (chunk == 0 && tid == 0) {
        s->klo = klo;
        s->khi = khi;
        s->c0 = c0;
        s->U = __builtin_inf();
        s->Ut = 0.0;
        s->zeros = zeros;
    }
    if (first < 0) return;
    const bool tied = __builtin_amdgcn_readfirstlane(sh.tied) != 0;
    HYRES_GLOBAL T* seg = gmem(static_cast<T*>(d.slist)) + comp * d.slcs + (int64_t)chunk * d.segcap;
    double s0 = 0.0;
    if (__builtin_expect(tied, 0)) {
        clear_ties(ties);
        __syncthreads();
        s0 = fold_ties<T>(cf + e0, e1 - e0, klo, khi, ties, [fine](typename KT::K k) { return first_bin<T>(k, fine); },
                          seg, (uint32_t)d.segcap, &sh.count);
    } else {
        for (int64_t e = e0 + tid - lane; e < e1; e += U * kSureThreads) {   // whole waves
#pragma unroll
            for (int u = 0; u < U; ++u) {
                v[u] = e + lane + (int64_t)u * kSureThreads < e1 ? v[u] : (T)0;
                if (KT::key(v[u]) < klo) s0 = fma((double)v[u], (double)v[u], s0);
            }
            keep_range<T, U>(v, klo, khi, seg, (uint32_t)d.segcap, &sh.count);
            if (e + U * kSureThreads < e1) fetch(e + U * kSureThreads);
        }
    }
    s0 = wave_sum(s0);
    if (lane == 0) sh.ws[wave] = s0;
    __syncthreads();
    if (tied) {
        keep_ties<T>(ties, seg + d.segcap, d.segcap, &sh.pairs);
        __syncthreads();
    }
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < kSureWaves; ++w) s += sh.ws[w];
        SureSeg* o = d.sseg + (int64_t)comp * d.snch + chunk;
        o->s0 = s;
        o->count = sh.count;
        o->pairs = sh.pairs;
    }
}

// Select on a histogram of counts c and sums of squares q (bins 4 tid + j, 2^shf keys
// wide) of the range [klo, khi), with c0 values and squares s0 below it: the values
// and squares before each thread's bins, the lower bounds of the bins and the
// smallest upper bound with its threshold.
template <typename T>
__device__ __forceinline__ void range_select(const uint32_t (&c)[kBinsPer], const double (&q)[kBinsPer], double N,
                                             uint64_t klo, uint64_t khi, int shf, uint64_t c0, double s0,
                                             SureShared& sh, uint32_t* before, double* sbefore,
                                             double (&lb)[kBinsPer], double* us, double* ut) {
    typedef KeyTraits<T> KT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t tc = 0;
    double tq = 0.0;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j) {
        tc += c[j];
        tq += q[j];
    }
    const uint32_t ic = wave_incl_u32(tc);
    const double iq = wave_incl_f64(tq), pq = __shfl_up(iq, 1, 64);
    if (lane == 63) {
        sh.wc[wave] = ic;
        sh.ws[wave] = iq;
    }
    __syncthreads();
    uint32_t total;
    double all;
    uint32_t pc = waves_before(sh.wc, wave, &total) + ic - tc;
    double ps = waves_before(sh.ws, wave, &all);
    if (lane) ps += pq;
    *before = pc;
    *sbefore = ps;
    *us = __builtin_inf();
    *ut = 0.0;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j) {
        const int b = kBinsPer * tid + j;
        lb[j] = __builtin_inf();
        if (c[j]) {
            const double C = (double)(c0 + pc), S = s0 + ps, cc = (double)c[j];
            const uint64_t end = klo + ((uint64_t)(b + 1) << shf);
            const double t0 = KT::val(klo + ((uint64_t)b << shf)), t1 = KT::val((end < khi ? end : khi) - 1);
            lb[j] = N - 2.0 * (C + cc) + S + (N - C) * t0 * t0;
            const double up = N - 2.0 * (C + cc) + (S + q[j]) + (N - C - cc) * t1 * t1;
            if (up < *us || (up == *us && t1 < *ut)) {
                *us = up;
                *ut = t1;
            }
        }
        pc += c[j];
        ps += q[j];
    }
}

// Argmin over the block of each thread's (s, t), smaller t on ties, to every thread.
__device__ __forceinline__ void block_argmin(double& s, double& t, SureShared& sh) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_argmin(s, t);
    __syncthreads();
    if (lane == 0) {
        sh.bs[wave] = s;
        sh.bt[wave] = t;
    }
    __syncthreads();
    s = sh.bs[lane & 15];
    t = sh.bt[lane & 15];
    wave_argmin(s, t);
}

// ---- large components: the range narrowed by all blocks before the finish ----
// (its list grows with the component, about 4 % of the values and an eighth of that a
// round later, and the one block reads it several times: of 67 million values the
// search took 2.8 ms, 2.35 of them the finish; 0.31 with two rounds)

// Values of a list, of a segment or of a chunk, and pairs of value and count, which
// lie downwards from `end`.
template <typename T>
struct SurePart {
    const HYRES_GLOBAL T* p;
    int64_t m;
    const HYRES_GLOBAL T* end;
    int pairs;
};
template <typename T>
__device__ __forceinline__ SurePart<T> sure_chunk_part(const CubeDesc& d, int comp, int chunk) {
    const int64_t e0 = (int64_t)chunk * d.schunk;
    return {gmem(static_cast<const T*>(d.coef)) + (int64_t)comp * d.ncs + e0, min(d.schunk, sure_count(d) - e0), nullptr, 0};
}
// Values and pairs that fit a list's space of `cap`
__device__ __forceinline__ bool sure_fits(uint32_t count, uint32_t pairs, int64_t cap) {
    return (int64_t)count + 2 * (int64_t)pairs <= cap;
}
// The gather's: a chunk's segment, or the chunk itself where the segment overflowed.
template <typename T>
__device__ __forceinline__ SurePart<T> sure_segment(const CubeDesc& d, int comp, int chunk, uint32_t count, uint32_t pairs) {
    if (!sure_fits(count, pairs, d.segcap)) return sure_chunk_part<T>(d, comp, chunk);
    const HYRES_GLOBAL T* seg = gmem(static_cast<const T*>(d.slist)) + comp * d.slcs + (int64_t)chunk * d.segcap;
    return {seg, (int64_t)count, seg + d.segcap, (int)pairs};
}
// A round's: one list per component, in the halves of its space in turn (the
// segments are in the first).
template <typename T>
__device__ __forceinline__ HYRES_GLOBAL T* sure_list(const CubeDesc& d, int comp, int round) {
    return gmem(static_cast<T*>(d.slist)) + comp * d.slcs + (round & 1 ? d.segcap * d.snch : 0);
}
// Values and pairs that a block of round `round` takes.
template <typename T>
__device__ __forceinline__ SurePart<T> sure_share(const CubeDesc& d, int comp, int chunk, int round, uint32_t count,
                                                  uint32_t pairs) {
    if (round == 0) {
        const SureSeg* g = d.sseg + (int64_t)comp * d.snch + chunk;
        return sure_segment<T>(d, comp, chunk, g->count, g->pairs);
    }
    const int64_t cap = d.segcap * d.snch;
    if (!sure_fits(count, pairs, cap)) return sure_chunk_part<T>(d, comp, chunk);
    const int64_t per = ((int64_t)count + d.snch - 1) / d.snch, a = min(chunk * per, (int64_t)count);
    const int64_t pp = ((int64_t)pairs + d.snch - 1) / d.snch, b = min(chunk * pp, (int64_t)pairs);
    const HYRES_GLOBAL T* list = sure_list<T>(d, comp, round);
    return {list + a, min(per, (int64_t)count - a), list + cap - 2 * b, (int)min(pp, (int64_t)pairs - b)};
}
// Row of counts and row of sums of squares of round `round`, behind the count rows.
__device__ __forceinline__ HYRES_GLOBAL uint32_t* refine_counts(const CubeDesc& d, int comp, int round) {
    return gmem(d.shist) + comp * d.shcs + (int64_t)(d.snch + 1 + 3 * round) * kSureBins;
}
__device__ __forceinline__ HYRES_GLOBAL double* refine_sums(const CubeDesc& d, int comp, int round) {
    return (HYRES_GLOBAL double*)(refine_counts(d, comp, round) + kSureBins);
}

// Histogram of counts and sums of squares over the range, added to the component's rows.
template <typename T>
__global__ __launch_bounds__(kSureThreads) void k_sure_refine(const CubeDesc* __restrict__ descs,
                                                              const int* __restrict__ items, int ncubes, int round) {
    typedef KeyTraits<T> KT;
    __shared__ uint32_t cnt[kSureBins];
    __shared__ double sum[kSureBins];
    const int cu = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[cu];
    const int nch = d.snch, local = blockIdx.x - items[cu], comp = local / nch, chunk = local - comp * nch;
    const int tid = threadIdx.x;
    if (round >= d.srounds) return;
    const SureSel s = d.ssel[comp * (d.srounds + 1) + round];
    if (s.khi <= s.klo) return;
    for (int b = tid; b < kSureBins; b += kSureThreads) {
        cnt[b] = 0;
        sum[b] = 0.0;
    }
    __syncthreads();
    const SurePart<T> a = sure_share<T>(d, comp, chunk, round, s.count, s.pairs);
    const int shf = shift_for(s.khi - s.klo);
    constexpr int U = kSureLoads;
    for (int64_t e = tid; e < a.m; e += U * kSureThreads) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = e + (int64_t)u * kSureThreads;
            v[u] = a.p[i < a.m ? i : a.m - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t k = KT::key(v[u]);
            if (e + (int64_t)u * kSureThreads < a.m && k >= s.klo && k < s.khi) {
                const int b = (int)((k - s.klo) >> shf);
                atomicAdd(&cnt[b], 1u);
                atomicAdd(&sum[b], (double)v[u] * (double)v[u]);
            }
        }
    }
    for (int e = tid; e < a.pairs; e += kSureThreads) {
        const double v = a.end[-2 * e - 2], n = a.end[-2 * e - 1];
        const uint64_t k = KT::key((T)v);
        if (k >= s.klo && k < s.khi) {
            const int b = (int)((k - s.klo) >> shf);
            atomicAdd(&cnt[b], (uint32_t)n);
            atomicAdd(&sum[b], n * (v * v));
        }
    }
    __syncthreads();
    HYRES_GLOBAL uint32_t* gc = refine_counts(d, comp, round);
    HYRES_GLOBAL double* gs = refine_sums(d, comp, round);
    for (int b = tid; b < kSureBins; b += kSureThreads)
        if (cnt[b]) {
            atomicAdd(&gc[b], cnt[b]);
            atomicAdd(&gs[b], sum[b]);
        }
}

// Select on those rows by every block, then the chunk's values in the narrower range.
template <typename T>
__global__ __launch_bounds__(kSureThreads) void k_sure_narrow(const CubeDesc* __restrict__ descs,
                                                              const int* __restrict__ items, int ncubes, int round) {
    typedef KeyTraits<T> KT;
    __shared__ SureShared sh;
    __shared__ SureTies<T> ties;
    const int cu = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[cu];
    const int nch = d.snch, local = blockIdx.x - items[cu], comp = local / nch, chunk = local - comp * nch;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (round >= d.srounds) return;
    const SureSel* s = d.ssel + comp * (d.srounds + 1) + round;
    const uint64_t klo = s->klo, khi = s->khi, c0 = s->c0;
    SureSel* o = d.ssel + comp * (d.srounds + 1) + round + 1;     // written by the first chunk's block, read by the next launch
    if (khi <= klo) {
        if (chunk == 0 && tid == 0) {
            o->klo = o->khi = 1;
            o->U = s->U;
            o->Ut = s->Ut;
            o->zeros = s->zeros;
        }
        return;
    }
    const double N = (double)sure_count(d);
    const SureSeg* sg = d.sseg + (int64_t)comp * d.snch;
    double s0 = 0.0;
    if (round == 0) {
        // squares below the range: lane sums of every 64th chunk, the same in every wave
        for (int k = lane; k < nch; k += 64) s0 += sg[k].s0;
        s0 = wave_sum(s0);
    } else {
        s0 = s->s0;
    }
    uint32_t c[kBinsPer], pc;
    double q[kBinsPer], lb[kBinsPer], ps, us, ut;
    const HYRES_GLOBAL uint32_t* gc = refine_counts(d, comp, round) + kBinsPer * tid;
    const HYRES_GLOBAL double* gs = refine_sums(d, comp, round) + kBinsPer * tid;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j) {
        c[j] = gc[j];
        q[j] = gs[j];
    }
    const int shf = shift_for(khi - klo);
    range_select<T>(c, q, N, klo, khi, shf, c0, s0, sh, &pc, &ps, lb, &us, &ut);
    block_argmin(us, ut, sh);
    double U = s->U, Ut = s->Ut;
    if (us < U) {
        U = us;
        Ut = ut;
    }
    const double U0 = fmin(U, N - 2.0 * (double)s->zeros), lim = U0 + 1e-12 * (fabs(U0) + N);
    int f = 0x7fffffff, l = -1;
#pragma unroll
    for (int j = 0; j < kBinsPer; ++j)
        if (lb[j] <= lim) {
            const int b = kBinsPer * tid + j;
            f = b < f ? b : f;
            l = b;
        }
    const int wf = wave_minmax_i32<false>(f), wl = wave_minmax_i32<true>(l);
    __syncthreads();
    if (lane == 63) {
        sh.wf[wave] = wf;
        sh.wl[wave] = wl;
    }
    if (tid == 0) sh.tied = 0;
    __syncthreads();
    f = waves_minmax<false>(sh.wf);
    l = waves_minmax<true>(sh.wl);
    if (bins_tied(c, f, l)) sh.tied = 1;
    __syncthreads();
    uint64_t nlo = 1, nhi = 1;
    if (l >= 0) {
        const uint64_t end = klo + ((uint64_t)(l + 1) << shf);
        nlo = klo + ((uint64_t)f << shf);
        nhi = end < khi ? end : khi;
    }
    if (chunk == 0) {
        if (tid == (l >= 0 ? f / kBinsPer : 0)) {
            uint64_t cf = c0 + pc;
            double sf = s0 + ps;
#pragma unroll
            for (int j = 0; j < kBinsPer; ++j)
                if (l >= 0 && kBinsPer * tid + j < f) {
                    cf += c[j];
                    sf += q[j];
                }
            o->klo = nlo;
            o->khi = nhi;
            o->c0 = cf;
            o->s0 = sf;
            o->U = U;
            o->Ut = Ut;
            o->zeros = s->zeros;
        }
    }
    if (l < 0) return;
    const SurePart<T> a = sure_share<T>(d, comp, chunk, round, s->count, s->pairs);
    HYRES_GLOBAL T* list = sure_list<T>(d, comp, round + 1);
    const int64_t cap = d.segcap * nch;
    const bool tied = __builtin_amdgcn_readfirstlane(sh.tied) != 0;
    if (__builtin_expect(tied, 0)) {
        clear_ties(ties);
        __syncthreads();
        (void)fold_ties<T>(a.p, a.m, nlo, nhi, ties, [&](typename KT::K k) { return (int)(((uint64_t)k - klo) >> shf); },
                           list, (uint32_t)cap, &o->count);
    } else {
        constexpr int V = kSureLoads;
        for (int64_t e = tid - lane; e < a.m; e += V * kSureThreads) {     // whole waves
            T v[V];
#pragma unroll
            for (int u = 0; u < V; ++u) {
                const int64_t i = e + lane + (int64_t)u * kSureThreads;
                v[u] = a.p[i < a.m ? i : a.m - 1];
            }
#pragma unroll
            for (int u = 0; u < V; ++u) v[u] = e + lane + (int64_t)u * kSureThreads < a.m ? v[u] : (T)0;
            keep_range<T, V>(v, nlo, nhi, list, (uint32_t)cap, &o->count);
        }
    }
    for (int e = tid; e < a.pairs; e += kSureThreads) {
        const T v = a.end[-2 * e - 2], n = a.end[-2 * e - 1];
        const uint64_t k = KT::key(v);
        if (k >= nlo && k < nhi) {
            const int64_t at = 2 * (int64_t)(atomicAdd(&o->pairs, 1u) + 1u);
            if (at <= cap) {
                list[cap - at] = v;
                list[cap - at + 1] = n;
            }
        }
    }
    if (tied) {
        __syncthreads();
        keep_ties<T>(ties, list + cap, cap, &o->pairs);
    }
}

// A range of keys to search: values and squares below it, a lower bound.
struct SureRange {
    uint64_t klo, khi, c0;
    double s0, lb;
};

template <typename T>
__global__ __launch_bounds__(kSureThreads) void k_sure_finish(const CubeDesc* __restrict__ descs,
                                                              const int* __restrict__ items, int ncubes) {
    typedef KeyTraits<T> KT;
    typedef typename KT::K K;
    constexpr int PER = kBinsPer, CAP = KT::kCap;
    __shared__ uint32_t cnt[kSureBins];       // values per bin
    __shared__ uint32_t pre[kSureBins];       // ... below the bin
    __shared__ uint32_t off[kSureBins];       // end of the bin's values in `keys`
    __shared__ double sum[kSureBins];         // squares per bin, then below the bin
    __shared__ K keys[CAP];
    __shared__ uint32_t bits[kSureBins / 32];
    __shared__ SureRange stack[kSureStack];
    __shared__ SureShared sh;
    __shared__ int s_sp, s_inexact, s_wlo[kSureWindows], s_whi[kSureWindows];
    __shared__ uint32_t s_count[kSureChunks], s_pairs[kSureChunks];
    const int cu = find_cube(items, ncubes, blockIdx.x);
    const CubeDesc& d = descs[cu];
    const int comp = blockIdx.x - items[cu];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t Ni = sure_count(d);
    const double N = (double)Ni;
    const int nch = d.snch;
    const HYRES_GLOBAL T* coef = gmem(static_cast<const T*>(d.coef)) + (int64_t)comp * d.ncs;
    // f(value, how often) for each of the values: the coefficients, or the list of the
    // last round, taken by the whole block; or the chunks' segments, in parts that
    // the waves take in turn.
    SurePart<T> whole = {coef, Ni, nullptr, 0};
    const int parts = (kSureWaves + nch - 1) / nch;
    auto run = [&](auto loads, const HYRES_GLOBAL T* p, int64_t a, int64_t b, int stride, auto f) {
        constexpr int U = decltype(loads)::value;
        for (int64_t i = a; i < b; i += (int64_t)stride * U) {
            T v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int64_t e = i + (int64_t)stride * k;
                v[k] = e < b ? p[e] : (T)0;           // few of the U are in range: clamped loads are slower here (40.3 us, 38)
            }
#pragma unroll
            for (int k = 0; k < U; ++k) f(v[k], 1u);      // zeros are in no range
        }
    };
    auto run_pairs = [&](const SurePart<T>& q, int a, int stride, auto f) {
        for (int i = a; i < q.pairs; i += stride) f(q.end[-2 * i - 2], (uint32_t)q.end[-2 * i - 1]);
    };
    auto for_each = [&](auto pairs, auto f) {
        const std::integral_constant<int, decltype(pairs)::value ? 4 : kSureLoads> loads{};   // (few values beside pairs)
        if (whole.p) {
            run(loads, whole.p, tid, whole.m, kSureThreads, f);
            if constexpr (decltype(pairs)::value) run_pairs(whole, tid, kSureThreads, f);
            return;
        }
        for (int u = wave; u < nch * parts; u += kSureWaves) {
            const int s = u / parts, part = u - s * parts;
            const SurePart<T> q = sure_segment<T>(d, comp, s, s_count[s], s_pairs[s]);
            const int64_t step = (q.m + parts - 1) / parts, a = part * step, b = min(a + step, q.m);
            run(loads, q.p, a + lane, b, 64, f);
            if constexpr (decltype(pairs)::value)
                if (part == 0) run_pairs(q, lane, 64, f);
        }
    };

    uint32_t zeros = 0;
    uint64_t klo = 1, khi = 1, c0 = 0;
    double s0 = 0.0, U = __builtin_inf(), Ut = 0.0;
    int64_t visits = 0;                       // values read so far
    bool need_s0 = false;
    if (nch == 1) {
        for (int b = tid; b < kSureBins; b += kSureThreads) cnt[b] = 0;
        __syncthreads();
        const uint32_t nz = first_histogram<T>(coef, 0, Ni, KT::kFine, cnt);
        if (nz) atomicAdd(&cnt[kZeroSlot], nz);
        __syncthreads();
        uint32_t c[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) c[j] = cnt[PER * tid + j];
        zeros = cnt[kZeroSlot];
        if (tid == kSureThreads - 1) c[PER - 1] = 0;
        int first, last;
        first_select<T, false>(c, zeros, N, KT::kFine, sh, &first, &last, &c0);
        if (first >= 0) first_range<T>(first, last, KT::kFine, &klo, &khi);
        need_s0 = true;
    } else {
        const SureSel s = d.ssel[comp * (d.srounds + 1) + d.srounds];
        klo = s.klo;
        khi = s.khi;
        c0 = s.c0;
        zeros = s.zeros;
        U = s.U;
        Ut = s.Ut;
        if (d.srounds) {
            s0 = s.s0;
            const HYRES_GLOBAL T* list = sure_list<T>(d, comp, d.srounds);
            const uint32_t count = readlane_u32(s.count, 0), pairs = readlane_u32(s.pairs, 0);
            if (sure_fits(count, pairs, d.segcap * nch))
                whole = {list, (int64_t)count, list + d.segcap * nch, (int)pairs};
        } else {
            whole.p = nullptr;
            const SureSeg* sg = d.sseg + (int64_t)comp * d.snch;
            if (khi > klo) {
                static_assert(kSureChunks == 64, "a lane per chunk");
                const SureSeg g = sg[lane < nch ? lane : 0];
                if (tid < nch) {
                    s_count[tid] = g.count;
                    s_pairs[tid] = g.pairs;
                    sum[tid] = g.s0;
                }
                whole.m = readlane_u32(wave_incl_u32(lane < nch ? min(g.count, (uint32_t)d.schunk) : 0u), 63);
                whole.pairs = (int)readlane_u32(wave_incl_u32(lane < nch ? g.pairs : 0u), 63);
                __syncthreads();
#pragma unroll 8
                for (int k = 0; k < nch; ++k) s0 += sum[k];
            }
        }
    }
    // candidate 0 and the smallest upper bound so far
    double best_s = N - 2.0 * (double)zeros, best_t = 0.0;
    if (best_s <= U) {
        U = best_s;
        Ut = 0.0;
    }
    if (tid == 0) {
        s_sp = 0;
        s_inexact = 0;
        if (khi > klo) {
            stack[0].klo = klo;
            stack[0].khi = khi;
            stack[0].c0 = c0;
            stack[0].s0 = s0;
            stack[0].lb = -__builtin_inf();
            s_sp = 1;
        }
    }
    __syncthreads();
    // (without pairs, as most components are, the code of their loops is out of the way)
    auto search = [&](auto pairs) {
        while (true) {
            __syncthreads();
            const int sp = s_sp;
            if (sp == 0) break;
            klo = stack[sp - 1].klo;
            khi = stack[sp - 1].khi;
            c0 = stack[sp - 1].c0;
            s0 = stack[sp - 1].s0;
            const double tol = 1e-12 * (fabs(U) + N);
            const bool skip = !(stack[sp - 1].lb <= U + tol);
            __syncthreads();
            if (tid == 0) s_sp = sp - 1;
            if (skip) continue;
            if (visits + whole.m + whole.pairs > kSureVisits) {
                if (tid == 0) {
                    s_inexact = 1;
                    s_sp = 0;
                }
                continue;
            }
            visits += whole.m + whole.pairs;
            const int shf = shift_for(khi - klo);
            for (int b = tid; b < kSureBins; b += kSureThreads) {
                cnt[b] = 0;
                sum[b] = 0.0;
            }
            __syncthreads();
            double below = 0.0;
            for_each(pairs, [&](T v, uint32_t n) {
                const uint64_t k = KT::key(v);
                if (k >= klo && k < khi) {
                    const int b = (int)((k - klo) >> shf);
                    atomicAdd(&cnt[b], n);
                    atomicAdd(&sum[b], (double)n * ((double)v * (double)v));
                } else if (need_s0 && k < klo) {
                    below = fma((double)v, (double)v, below);
                }
            });
            if (need_s0) {
                below = wave_sum(below);
                if (lane == 0) sh.ws[wave] = below;
            }
            __syncthreads();
            if (need_s0) {
                (void)waves_before(sh.ws, wave, &s0);
                need_s0 = false;
                __syncthreads();
            }
            uint32_t c[PER], pc;
            double q[PER], lb[PER], ps, us, ut;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                c[j] = cnt[PER * tid + j];
                q[j] = sum[PER * tid + j];
            }
            range_select<T>(c, q, N, klo, khi, shf, c0, s0, sh, &pc, &ps, lb, &us, &ut);
#pragma unroll
            for (int j = 0; j < PER; ++j) {       // exclusive prefixes
                pre[PER * tid + j] = pc;
                sum[PER * tid + j] = ps;
                pc += c[j];
                ps += q[j];
            }
            block_argmin(us, ut, sh);
            if (us < U) {
                U = us;
                Ut = ut;
            }
            if (shf == 0) {                       // one value per bin: the bounds are exact
                if (us < best_s || (us == best_s && ut < best_t)) {
                    best_s = us;
                    best_t = ut;
                }
                continue;
            }
            const double lim = U + 1e-12 * (fabs(U) + N);
            int f = 0x7fffffff, l = -1, mx = 0, nh = 0;
            uint32_t m = 0, ml = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (lb[j] <= lim) {
                    const int b = PER * tid + j, n = c[j] < 0x7fffffffu ? (int)c[j] : 0x7fffffff;
                    f = b < f ? b : f;
                    l = b;
                    mx = n > mx ? n : mx;
                    nh += n > kSureHeavy ? 1 : 0;
                    m += c[j];
                    ml += n > kSureHeavy ? 0 : c[j];
                }
            const int wf = wave_minmax_i32<false>(f), wl = wave_minmax_i32<true>(l), wx = wave_minmax_i32<true>(mx);
            const uint32_t wm = wave_incl_u32(m), wh = wave_incl_u32((uint32_t)nh), wlt = wave_incl_u32(ml);
            __syncthreads();
            if (lane == 63) {
                sh.wf[wave] = wf;
                sh.wl[wave] = wl;
                sh.wx[wave] = wx;
                sh.wc[wave] = wm;
                sh.wn[wave] = wh;
                sh.wm[wave] = wlt;
            }
            __syncthreads();
            f = waves_minmax<false>(sh.wf);
            l = waves_minmax<true>(sh.wl);
            mx = waves_minmax<true>(sh.wx);
            uint32_t total, heavies, light;
            (void)waves_before(sh.wc, wave, &total);
            (void)waves_before(sh.wn, wave, &heavies);
            (void)waves_before(sh.wm, wave, &light);
            if (l < 0) continue;
            if ((total > (uint32_t)CAP || mx > kSureLight) && (l - f + 1) * 2 <= kSureBins) {
                // the surviving bins span at most half the range: search that
                if (tid == 0) {
                    const uint64_t hi = klo + ((uint64_t)(l + 1) << shf);
                    SureRange& r = stack[s_sp];
                    r.klo = klo + ((uint64_t)f << shf);
                    r.khi = hi < khi ? hi : khi;
                    r.c0 = c0 + pre[f];
                    r.s0 = s0 + sum[f];
                    r.lb = -__builtin_inf();
                    s_sp = s_sp + 1;
                }
                continue;
            }
            if (light > (uint32_t)CAP || heavies > (uint32_t)kSureHeavies) {
                // flat over more than half the range: windows of it, each a range with bins as
                // many times finer, down to about a sixteenth of the values
                const int span = l - f + 1;
                const int nw = (int)min((uint32_t)kSureWindows, total / (4u * CAP) + 2u);
                if (tid < kSureWindows) {
                    s_wlo[tid] = kSureBins;
                    s_whi[tid] = -1;
                }
                __syncthreads();
#pragma unroll
                for (int j = 0; j < PER; ++j)
                    if (lb[j] <= lim) {
                        const int b = PER * tid + j, w = (b - f) * nw / span;
                        atomicMin(&s_wlo[w], b);
                        atomicMax(&s_whi[w], b);
                    }
                __syncthreads();
                if (tid < nw && s_whi[tid] >= 0) {
                    const int at = atomicAdd(&s_sp, 1), b0 = s_wlo[tid], b1 = s_whi[tid];
                    if (at < kSureStack) {
                        const uint64_t hi = klo + ((uint64_t)(b1 + 1) << shf);
                        SureRange& r = stack[at];
                        r.klo = klo + ((uint64_t)b0 << shf);
                        r.khi = hi < khi ? hi : khi;
                        r.c0 = c0 + pre[b0];
                        r.s0 = s0 + sum[b0];
                        r.lb = -__builtin_inf();
                    } else {
                        s_inexact = 1;
                    }
                }
                __syncthreads();
                if (tid == 0 && s_sp > kSureStack) s_sp = kSureStack;
                continue;
            }
            // bins too large to evaluate value by value become ranges of their own
            uint32_t g[PER], tg = 0;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int b = PER * tid + j;
                g[j] = 0;
                if (!(lb[j] <= lim)) continue;
                if (c[j] > (uint32_t)kSureHeavy) {
                    const int at = atomicAdd(&s_sp, 1);
                    if (at < kSureStack) {
                        const uint64_t hi = klo + ((uint64_t)(b + 1) << shf);
                        SureRange& r = stack[at];
                        r.klo = klo + ((uint64_t)b << shf);
                        r.khi = hi < khi ? hi : khi;
                        r.c0 = c0 + pre[b];
                        r.s0 = s0 + sum[b];
                        r.lb = lb[j];
                    } else {
                        s_inexact = 1;
                    }
                } else {
                    g[j] = c[j];
                    tg += c[j];
                }
            }
            const uint32_t ig = wave_incl_u32(tg);
            __syncthreads();
            if (lane == 63) sh.wc[wave] = ig;
            if (tid == 0 && s_sp > kSureStack) s_sp = kSureStack;
            __syncthreads();
            const uint32_t og = waves_before(sh.wc, wave, &light) + ig - tg;
            if (light) {                          // at most CAP values
                if (tid < kSureBins / 32) bits[tid] = 0;
                __syncthreads();
                uint32_t o = og;
                uint32_t mine = 0;
#pragma unroll
                for (int j = 0; j < PER; ++j) {
                    if (g[j]) {
                        off[PER * tid + j] = o;
                        mine |= 1u << j;
                    }
                    o += g[j];
                }
                if (mine) atomicOr(&bits[tid >> 3], mine << (4 * (tid & 7)));
                __syncthreads();
                for_each(pairs, [&](T v, uint32_t n) {
                    const uint64_t k = KT::key(v);
                    if (k >= klo && k < khi) {
                        const int b = (int)((k - klo) >> shf);
                        if ((bits[b >> 5] >> (b & 31)) & 1u) {
                            const uint32_t at = atomicAdd(&off[b], n);
                            for (uint32_t i = 0; i < n; ++i) keys[at + i] = (K)k;
                        }
                    }
                });
                __syncthreads();
                double es = __builtin_inf(), et = 0.0;
                for (int i = tid; i < (int)light; i += kSureThreads) {
                    const uint64_t key = keys[i];
                    const int b = (int)((key - klo) >> shf);
                    const int n = (int)cnt[b], j1 = (int)off[b];
                    int in = 0;
                    double sq = 0.0;
                    for (int j = j1 - n; j < j1; j += 4) {      // four reads in flight, added in order
                        uint64_t kj[4];
#pragma unroll
                        for (int w = 0; w < 4; ++w) kj[w] = keys[j + w < j1 ? j + w : j1 - 1];
#pragma unroll
                        for (int w = 0; w < 4; ++w)
                            if (j + w < j1 && kj[w] <= key) {
                                const double vj = KT::val(kj[w]);
                                ++in;
                                sq = fma(vj, vj, sq);
                            }
                    }
                    const double cc = (double)(c0 + pre[b]) + (double)in, S = s0 + sum[b] + sq, v = KT::val(key);
                    const double sv = N - 2.0 * cc + S + (N - cc) * v * v;
                    if (sv < es || (sv == es && v < et)) {
                        es = sv;
                        et = v;
                    }
                }
                block_argmin(es, et, sh);
                if (es < best_s || (es == best_s && et < best_t)) {
                    best_s = es;
                    best_t = et;
                }
                if (best_s < U) U = best_s;
                __syncthreads();
            }
        }
    };
    if (__builtin_expect(whole.pairs == 0, 1)) search(std::integral_constant<bool, false>{});
    else search(std::integral_constant<bool, true>{});
    if (tid == 0) {
        if (s_inexact && U < best_s) {        // the end of a bin: no value of the component
            best_s = U;
            best_t = Ut;
        }
        d.lambda[comp] = best_t;
        if (d.sure) d.sure[comp] = best_s;
        if (s_inexact) set_status(d.status, HYRES_DEV_SURE_INEXACT);
    }
}

// ---------------------------------------------------------------- launchers
hipError_t launch_sure(int dtype, int step, const CubeDesc* descs, const int* items, int ncubes, int grid, int round,
                       hipStream_t s) {
#define HYRES_S(K, TH, ...)                                                                                   \
    if (dtype == HYRES_F64) hipLaunchKernelGGL(K<double>, dim3(grid), dim3(TH), 0, s, descs, items, ncubes __VA_ARGS__); \
    else hipLaunchKernelGGL(K<float>, dim3(grid), dim3(TH), 0, s, descs, items, ncubes __VA_ARGS__);           \
    break
    switch (step) {
        case SURE_HIST: HYRES_S(k_sure_hist, kSureThreads);
        case SURE_ROWS: HYRES_S(k_sure_rows, 256);
        case SURE_GATHER: HYRES_S(k_sure_gather, kSureThreads);
        case SURE_REFINE: HYRES_S(k_sure_refine, kSureThreads, , round);
        case SURE_NARROW: HYRES_S(k_sure_narrow, kSureThreads, , round);
        case SURE_FINISH: HYRES_S(k_sure_finish, kSureThreads);
        default: return hipErrorInvalidValue;
    }
#undef HYRES_S
    return hipGetLastError();
}

// Refining rounds before the finish.  The line lies where a round costs what it saves:
// one component of 2^20 values takes 75 us without and 65 with it, eight 82 and
// 85; of 2^21 values 109 and 82, 153 and 129; of 2^24 569 and 159.
int sure_rounds(int64_t N) {
    if (N <= kSureLarge) return 0;
    return N <= ((int64_t)1 << 24) ? 1 : N <= ((int64_t)1 << 28) ? 2 : kSureRefine;
}
// Words of the rows behind the count rows: the summed row and the refining rounds'.
int64_t sure_extra(int64_t N) { return N > kSureLarge ? (1 + 3 * kSureRefine) * (int64_t)kSureBins : 0; }

// Chunks of one component of N values in a program of `total` values: one per
// compute unit over all components, of at least 16384 values, at most those whose
// rows fit in `room` words and kSureChunks (kSureMaxChunks of a large component, whose
// rows a launch of their own adds up).  Components of up to kSureDirect values take one
// block for the whole search (two launches fewer; a block reads 65536 values in 2 us).
// Up to 64 chunks of 16-bit counts before longer ones.
int sure_chunks(int64_t N, int64_t total, int num_cu, int64_t room) {
    if (N <= kSureDirect) return 1;
    const int64_t most = N > kSureLarge ? kSureMaxChunks : kSureChunks;
    int64_t ch = (total + num_cu - 1) / num_cu;
    if (ch < 16384) ch = 16384;
    int64_t nch = (N + ch - 1) / ch;
    if (N <= 64 * kSureRow16 && (N + nch - 1) / nch > kSureRow16 - 1024) nch = (N + kSureRow16 - 1025) / (kSureRow16 - 1024);
    if (nch > most) nch = most;
    const int64_t rows = (room - sure_extra(N)) / kSureBins;
    if (nch > rows) nch = rows;
    return nch < 1 ? 1 : (int)nch;
}
int64_t sure_chunk(int64_t N, int nch) {
    return ((N + nch - 1) / nch + kSureThreads - 1) / kSureThreads * kSureThreads;
}

}  // namespace hyres
