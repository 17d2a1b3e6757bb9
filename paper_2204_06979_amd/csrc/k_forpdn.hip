// FORPDN (Section 2.1: full-rank, wavelet-based, first-order spectral
// roughness penalty, for Gaussian noise).  The cube is whitened by the
// per-band noise, transformed band by band with the periodised 2-D db2
// wavelet, and every coefficient vector (one position, all p bands) of a
// wavelet group (the details of one level, or the coarsest approximation) is
// replaced by (I + lam D^T D)^-1 c with the group's lam chosen by SURE.
//
// The bands of one position stay together from start to end (the cube is
// pixel-major; the coefficients are stored position-major, p contiguous
// values per position), so
//   k_vdwt_level   one analysis level: each thread computes the four subband
//                  values of 2 x 2 positions, 16 bytes of bands each, from one
//                  6 x 6 window; the first level scales by 1/sigma on load;
//   (the band Gram of each group is the pixel-major Gram kernel of HyRes run
//    on the group's positions as a "cube")
//   k_forpdn_lambda one block per group: the energies of the coefficient
//                  matrix in the DCT-II eigenbasis of D^T D from the group's
//                  Gram, then SURE of the smoother on the lam grid in closed
//                  form and its argmin;
//   k_forpdn_filter the tridiagonal solve of every coefficient vector (a row in
//                  the registers of one lane);
//   k_vidwt_level  one synthesis level; the last scales by sigma on store.
#include <algorithm>

#include "hyres_internal.hpp"

namespace hyres {

namespace {
constexpr double kG0 = kH3, kG1 = -kH2, kG2 = kH1, kG3 = -kH0;   // g[m] = (-1)^m h[3 - m]

// Sample i < 3 Ne of an axis of N samples, Ne = N rounded up to even: periodic,
// an odd length repeats its last sample.  A window starts at Ne - 2 at the latest
// and has six samples, Ne >= 2.
__device__ __forceinline__ int ext_index(int i, int N, int Ne) {
    i = i < Ne ? i : i - Ne;
    i = i < Ne ? i : i - Ne;
    return i == N ? N - 1 : i;
}

// V consecutive bands of one position.
template <typename T, int V> struct Bands { typedef T type __attribute__((ext_vector_type(V))); };
template <typename T> struct Bands<T, 1> { typedef T type; };
template <typename T, int V>
__device__ __forceinline__ void set_band(typename Bands<T, V>::type& v, int k, T x) {
    if constexpr (V == 1) v = x;
    else v[k] = x;
}

// Work item it of n as the it-th of an order in which each of the eight XCDs
// (blocks are dealt to them in turn) has a contiguous range: the rows that two
// neighbouring windows share are then read by the same XCD.
__device__ __forceinline__ int64_t xcd_item(int64_t it, int64_t n) {
    const int64_t x = it & 7, k = it >> 3;
    return x * (n >> 3) + (x < (n & 7) ? x : (n & 7)) + k;
}
// Walk over the positions of a bh x bw grid in strips of kStrip columns, row by
// row within a strip: the rows that neighbouring windows share come again after
// one strip's row (0.15 MB a row of four subbands at 144 bands), while they are
// still in the XCD's L2, instead of after a whole row.
constexpr int kStrip = 32;      // (64 measures the same)
struct Walk {
    int bh, bw, y, x, x0, sw;          // position (y, x0 + x) of the strip [x0, x0 + sw)
    __device__ __forceinline__ Walk(int bh_, int bw_, int64_t q) : bh(bh_), bw(bw_) {
        const int64_t st = q / ((int64_t)kStrip * bh);
        const int64_t r = q - st * kStrip * bh;
        x0 = (int)st * kStrip;
        sw = bw - x0 < kStrip ? bw - x0 : kStrip;
        y = (int)(r / sw);
        x = (int)(r - (int64_t)y * sw);
    }
    __device__ __forceinline__ void step(int n) {
        x += n;
        while (x >= sw) {
            x -= sw;
            if (++y == bh) {
                y = 0;
                x0 += kStrip;
                sw = bw - x0 < kStrip ? bw - x0 : kStrip;
            }
        }
    }
};
}  // namespace

// One analysis level.  A thread computes a 2 x 2 block of output positions of V
// consecutive bands (16 bytes where the layout allows): the 6 x 6 input window is
// read once (9 loads per position instead of 16).  The floor is one read and one
// write of the level; with 16-byte accesses, no 64-bit division per element and
// the scales in LDS the four levels of 349 x 1905 x 144 take 210 us, against
// 480 with one band per thread, whose address arithmetic bounded it.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_vdwt_level(VLevel a) {
    typedef typename Bands<T, V>::type VT;
    __shared__ T s_sc[kMaxBands];
    const T hf[4] = {(T)kH0, (T)kH1, (T)kH2, (T)kH3};
    const T gf[4] = {(T)kG0, (T)kG1, (T)kG2, (T)kG3};
    const int p = a.p, pv = p / V;
    const uint32_t mag = (uint32_t)((1ull << 32) / (uint32_t)pv + 1);
    const int Hext = a.Hin + (a.Hin & 1), Wext = a.Win + (a.Win & 1);
    const int bh = (a.h + 1) / 2, bw = (a.w + 1) / 2;         // 2 x 2 blocks of outputs
    const int64_t nq = (int64_t)bh * bw;
    const int64_t nitem = (nq * pv + 255) / 256;
    const int64_t sub = (int64_t)a.h * a.w * p;              // one detail block
    for (int b = threadIdx.x; b < p; b += 256) s_sc[b] = a.scale ? (T)(1.0 / a.scale[b]) : (T)1;
    __syncthreads();
    const HYRES_GLOBAL T* src = gmem(static_cast<const T*>(a.in));
    for (int64_t it = blockIdx.x; it < nitem; it += gridDim.x) {
        const int64_t e0 = xcd_item(it, nitem) * 256;
        const int64_t q0 = e0 / pv;
        Walk at(bh, bw, q0);
        const int e = (int)(e0 - q0 * pv) + threadIdx.x;
        if (e0 + threadIdx.x < nq * pv) {
            const int ql = pv == 1 ? e : (int)__umulhi((uint32_t)e, mag);   // e / pv
            const int b = (e - ql * pv) * V;
            at.step(ql);
            const int y0 = 2 * at.y, x0 = 2 * (at.x0 + at.x);
            VT sc;
#pragma unroll
            for (int k = 0; k < V; ++k) set_band<T, V>(sc, k, s_sc[b + k]);
            const HYRES_GLOBAL T* in = src + b;
            int64_t cx[6];
#pragma unroll
            for (int c = 0; c < 6; ++c) cx[c] = (int64_t)ext_index(2 * x0 + c, a.Win, Wext) * a.ip;
            // along x first (two output columns), in tap order
            VT rl[6][2], rh[6][2];
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                const HYRES_GLOBAL T* row = in + (int64_t)ext_index(2 * y0 + r, a.Hin, Hext) * a.irow;
                VT v[6];
#pragma unroll
                for (int c = 0; c < 6; ++c) v[c] = *(const HYRES_GLOBAL VT*)(row + cx[c]) * sc;
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    rl[r][o] = hf[0] * v[2 * o] + hf[1] * v[2 * o + 1] + hf[2] * v[2 * o + 2] + hf[3] * v[2 * o + 3];
                    rh[r][o] = gf[0] * v[2 * o] + gf[1] * v[2 * o + 1] + gf[2] * v[2 * o + 2] + gf[3] * v[2 * o + 3];
                }
            }
#pragma unroll
            for (int oy = 0; oy < 2; ++oy) {
                const int y = y0 + oy;
#pragma unroll
                for (int ox = 0; ox < 2; ++ox) {
                    const int x = x0 + ox;
                    if (y < a.h && x < a.w) {
                        // rows 2 oy .. 2 oy + 3 of the window
                        const VT l0 = rl[2 * oy][ox], l1 = rl[2 * oy + 1][ox], l2 = rl[2 * oy + 2][ox], l3 = rl[2 * oy + 3][ox];
                        const VT h0 = rh[2 * oy][ox], h1 = rh[2 * oy + 1][ox], h2 = rh[2 * oy + 2][ox], h3 = rh[2 * oy + 3][ox];
                        const VT ll = hf[0] * l0 + hf[1] * l1 + hf[2] * l2 + hf[3] * l3;
                        const VT hl = gf[0] * l0 + gf[1] * l1 + gf[2] * l2 + gf[3] * l3;
                        const VT lh = hf[0] * h0 + hf[1] * h1 + hf[2] * h2 + hf[3] * h3;
                        const VT hh = gf[0] * h0 + gf[1] * h1 + gf[2] * h2 + gf[3] * h3;
                        const int64_t o = ((int64_t)y * a.w + x) * p + b;
                        HYRES_GLOBAL T* det = gmem(static_cast<T*>(a.det)) + o;
                        *(HYRES_GLOBAL VT*)(det) = lh;
                        *(HYRES_GLOBAL VT*)(det + sub) = hl;
                        *(HYRES_GLOBAL VT*)(det + 2 * sub) = hh;
                        *(HYRES_GLOBAL VT*)(gmem(static_cast<T*>(a.ll)) + o) = ll;
                    }
                }
            }
        }
    }
}

// One synthesis level.  A thread computes a 2 x 2 block of output pixels of V
// consecutive bands: pixels (2Y + py, 2X + px) all take the coefficients at rows Y
// and Y - 1 and columns X and X - 1 (mod the subband size), taps py, py + 2 and
// px, px + 2.  Four levels of 349 x 1905 x 144: 261 us, 450 with one band
// per thread.
template <typename T, int V>
__global__ __launch_bounds__(256) void k_vidwt_level(VSyn a) {
    typedef typename Bands<T, V>::type VT;
    __shared__ T s_sc[kMaxBands];
    const T hf[4] = {(T)kH0, (T)kH1, (T)kH2, (T)kH3};
    const T gf[4] = {(T)kG0, (T)kG1, (T)kG2, (T)kG3};
    const int p = a.p, pv = p / V;
    const uint32_t mag = (uint32_t)((1ull << 32) / (uint32_t)pv + 1);
    const int64_t nq = (int64_t)a.h * a.w;                   // one block per subband position
    const int64_t nitem = (nq * pv + 255) / 256;
    const HYRES_GLOBAL T* LL = gmem(static_cast<const T*>(a.ll));
    const HYRES_GLOBAL T* LH = gmem(static_cast<const T*>(a.det));
    const HYRES_GLOBAL T* HL = LH + nq * p;
    const HYRES_GLOBAL T* HH = HL + nq * p;
    if (a.scale)
        for (int b = threadIdx.x; b < p; b += 256) s_sc[b] = (T)a.scale[b];
    __syncthreads();
    for (int64_t it = blockIdx.x; it < nitem; it += gridDim.x) {
        const int64_t e0 = xcd_item(it, nitem) * 256;
        const int64_t q0 = e0 / pv;
        Walk pos(a.h, a.w, q0);
        const int e = (int)(e0 - q0 * pv) + threadIdx.x;
        if (e0 + threadIdx.x < nq * pv) {
            const int ql = pv == 1 ? e : (int)__umulhi((uint32_t)e, mag);
            const int b = (e - ql * pv) * V;
            pos.step(ql);
            const int Y = pos.y, X = pos.x0 + pos.x;
            const int Ym = Y == 0 ? a.h - 1 : Y - 1, Xm = X == 0 ? a.w - 1 : X - 1;
            const int64_t i00 = ((int64_t)Y * a.w + X) * p + b, i01 = ((int64_t)Y * a.w + Xm) * p + b;
            const int64_t i10 = ((int64_t)Ym * a.w + X) * p + b, i11 = ((int64_t)Ym * a.w + Xm) * p + b;
            auto at = [](const HYRES_GLOBAL T* s, int64_t i) { return *(const HYRES_GLOBAL VT*)(s + i); };
            // [row Y or Y - 1][column X or X - 1]
            const VT ll[2][2] = {{at(LL, i00), at(LL, i01)}, {at(LL, i10), at(LL, i11)}};
            const VT hl[2][2] = {{at(HL, i00), at(HL, i01)}, {at(HL, i10), at(HL, i11)}};
            const VT lh[2][2] = {{at(LH, i00), at(LH, i01)}, {at(LH, i10), at(LH, i11)}};
            const VT hh[2][2] = {{at(HH, i00), at(HH, i01)}, {at(HH, i10), at(HH, i11)}};
            VT sc;
#pragma unroll
            for (int k = 0; k < V; ++k) set_band<T, V>(sc, k, a.scale ? s_sc[b + k] : (T)1);
#pragma unroll
            for (int py = 0; py < 2; ++py) {
                const int iy = 2 * Y + py;
                if (iy >= a.Hin) continue;
                // along y first: lo_x from LL and HL, hi_x from LH and HH (taps py then py + 2)
                VT lo[2], hi[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    lo[c] = (hf[py] * ll[0][c] + gf[py] * hl[0][c]) + (hf[py + 2] * ll[1][c] + gf[py + 2] * hl[1][c]);
                    hi[c] = (hf[py] * lh[0][c] + gf[py] * hh[0][c]) + (hf[py + 2] * lh[1][c] + gf[py + 2] * hh[1][c]);
                }
#pragma unroll
                for (int px = 0; px < 2; ++px) {
                    const int ix = 2 * X + px;
                    if (ix >= a.Win) continue;
                    VT v = (hf[px] * lo[0] + gf[px] * hi[0]) + (hf[px + 2] * lo[1] + gf[px + 2] * hi[1]);
                    if (a.scale) v *= sc;
                    *(HYRES_GLOBAL VT*)(gmem(static_cast<T*>(a.out)) + (int64_t)iy * a.orow + (int64_t)ix * a.op + b) = v;
                }
            }
        }
    }
}

// One block per group: e_k = q_k^T G q_k in the DCT-II basis q_k(i) =
// n_k cos(pi k (2i + 1) / (2p)), formed from the sums of G along its
// anti-diagonals (A_s = sum_{r+c=s} G_rc) and diagonals (B_t = sum_{r-c=t} G_rc)
// by the product-to-sum identity, O(p^2) per group; then SURE of the smoother
// (I + lam D^T D)^-1 at unit noise on the grid lam = 10^(t/10), t = -40..40, in
// closed form, SURE(lam) = sum_k e_k (lam d_k / (1 + lam d_k))^2 - N p
// + 2 N sum_k 1 / (1 + lam d_k), d_k = 2 - 2 cos(pi k / p), and its argmin
// (the smallest lam among equal minima).  With given thresholds only SURE at them.
// The sums over a diagonal are split over LA or LB threads, those over the
// basis and the grid over eight lanes, added in order (52 us with one thread per
// sum, whose strided loads followed one another; 31 now).
__global__ __launch_bounds__(1024) void k_forpdn_lambda(FLambda a) {
    constexpr int NT = 1024, LA = 2, LB = 4;
    __shared__ double s_cos[4 * kMaxBands];       // cos(pi m / (2p)), m < 4p
    __shared__ double s_A[2 * kMaxBands], s_B[kMaxBands];   // anti-diagonal sums; diagonal sums for |t| (both signs)
    __shared__ double s_pa[LA][2 * kMaxBands], s_pb[LB][kMaxBands];
    __shared__ double s_e[kMaxBands], s_d[kMaxBands];
    __shared__ double s_sure[kForpdnGrid];
    const int j = blockIdx.x, t = threadIdx.x, p = a.p, P4 = 4 * p;
    const HYRES_GLOBAL double* G = gmem(a.G[j]);
    const double N = (double)a.count[j];
    for (int m = t; m < P4; m += NT) s_cos[m] = cos(M_PI * (double)m / (2.0 * p));
    // entries at(i0), at(i0 + step), .. up to i1, 18 loads in flight
    auto batch_sum = [&](int i0, int i1, int step, auto at) {
        double acc = 0.0;
        for (int i = i0; i <= i1; i += 18 * step) {
            double v[18];
#pragma unroll
            for (int u = 0; u < 18; ++u) v[u] = G[at(i + u * step <= i1 ? i + u * step : i1)];
#pragma unroll
            for (int u = 0; u < 18; ++u) acc += i + u * step <= i1 ? v[u] : 0.0;
        }
        return acc;
    };
    static_assert(2 * kMaxBands * LA <= NT && kMaxBands * LB <= NT, "one thread per partial sum");
    {
        const int sidx = t % (2 * kMaxBands), part = t / (2 * kMaxBands);
        if (part < LA && sidx < 2 * p - 1) {
            const int r0 = sidx < p ? 0 : sidx - p + 1, r1 = sidx < p ? sidx : p - 1;
            s_pa[part][sidx] = batch_sum(r0 + part, r1, LA, [&](int r) { return r * p + (sidx - r); });
        }
    }
    {
        const int d = t % kMaxBands, part = t / kMaxBands;
        if (part < LB && d < p) {
            const double acc = batch_sum(part, p - 1 - d, LB, [&](int c) { return c * p + (c + d); });
            s_pb[part][d] = d > 0 ? 2.0 * acc : acc;         // G is symmetric, both halves stored
        }
    }
    __syncthreads();
    for (int sidx = t; sidx < 2 * p - 1; sidx += NT) s_A[sidx] = s_pa[0][sidx] + s_pa[1][sidx];
    for (int d = t; d < p; d += NT) s_B[d] = (s_pb[0][d] + s_pb[1][d]) + (s_pb[2][d] + s_pb[3][d]);
    __syncthreads();
    // sum over the eight lanes of an aligned group, to every lane
    auto sum8 = [](double v) {
        v += dpp_f64<0xB1>(v);
        v += dpp_f64<0x4E>(v);
        return v + dpp_f64<0x141>(v);
    };
    const int l8 = t & 7;
    // q_k^T G q_k = n_k^2 / 2 (sum_s A_s cos(pi k (s + 1) / p) + sum_t B_t cos(pi k t / p))
    const double c0 = 1.0 / p, ck = 2.0 / p;
    for (int k0 = 0; k0 < p; k0 += NT / 8) {
        const int k = k0 + t / 8;
        double sa = 0.0, sb = 0.0;
        if (k < p) {
            const int dm = (16 * k) % P4;            // 2 k (s + 1) and 2 k d mod 4 p, step by step
            int m = (2 * k * (l8 + 1)) % P4;
            for (int sidx = l8; sidx < 2 * p - 1; sidx += 8) {
                sa = fma(s_A[sidx], s_cos[m], sa);
                m += dm;
                m = m < P4 ? m : m - P4;
            }
            m = (2 * k * l8) % P4;
            for (int d = l8; d < p; d += 8) {
                sb = fma(s_B[d], s_cos[m], sb);
                m += dm;
                m = m < P4 ? m : m - P4;
            }
        }
        sa = sum8(sa + sb);
        if (k < p && l8 == 0) {
            s_e[k] = 0.5 * (k == 0 ? c0 : ck) * sa;
            s_d[k] = 2.0 - 2.0 * s_cos[(2 * k) % P4];
        }
    }
    __syncthreads();
    // eight lanes per threshold
    auto sure_at = [&](double lam) {
        double res = 0.0, tr = 0.0;
        for (int k = l8; k < p; k += 8) {
            const double f = 1.0 / (1.0 + lam * s_d[k]);
            const double o = 1.0 - f;
            res = fma(s_e[k] * o, o, res);
            tr += f;
        }
        return sum8(res) - N * p + 2.0 * N * sum8(tr);
    };
    if (a.lambda_in) {
        const double lam = a.lambda_in[j], v = sure_at(lam);
        if (t == 0) {
            a.lambda[j] = lam;
            a.sure[j] = v;
        }
        return;
    }
    static_assert(kForpdnGrid * 8 <= NT, "one pass over the grid");
    {
        const int g = t / 8;
        const double v = sure_at(pow(10.0, (double)((g < kForpdnGrid ? g : 0) - kForpdnGrid / 2) / 10.0));
        if (g < kForpdnGrid && l8 == 0) s_sure[g] = v;
    }
    __syncthreads();
    if (t == 0) {
        int best = 0;
        for (int g = 1; g < kForpdnGrid; ++g)
            if (s_sure[g] < s_sure[best]) best = g;
        a.lambda[j] = pow(10.0, (double)(best - kForpdnGrid / 2) / 10.0);
        a.sure[j] = s_sure[best];
    }
}

// Each lane owns one coefficient vector (a position) and keeps it in registers:
// a wave loads its 64 positions at once (16 bytes a lane, 16 bands of a row by
// neighbouring lanes), turns 16 bands at a time through a small LDS tile, solves
// (I + lam_j D^T D) x = c by Thomas' recurrence with the factors of all groups
// in LDS (formed in FP64 once per block), and writes the rows back the same way.
// The floor is one read and one write of the coefficients.  Rows kept whole in
// LDS left room for three waves on a compute unit, too few for the loads to
// overlap the recurrences: 349 x 1905 x 144 took 371 us, 160 us now.  A row and an
// address for each of its loads did not fit: 256 x 256 positions of 103 bands in
// FP32 took 48 us with 146 registers spilled (23 now, 42 with rows in LDS), of
// 191 97 (38, 121).  FP64 rows of more than 160 bands still spill (64 to 750
// bytes a lane; 224 bands 100 us, 238 with rows in LDS).
// The LDS rows of 16 bands are 20 (FP64 18) values apart: 16-byte accesses of 16
// neighbouring lanes then fall on different banks, by row and by column.
// NC chunks of 16 bands hold p; V bands per load (16 bytes if p allows, else one).
constexpr int kFWaves = 4;
template <typename T> constexpr int kFStride = sizeof(T) == 8 ? 18 : 20;
inline size_t filter_lds(int es, int nc, int groups) {
    const size_t tab = (size_t)2 * groups * nc * 16 * es;
    return tab + std::max((size_t)kFWaves * 64 * (es == 8 ? 18 : 20) * es, (size_t)groups * nc * 16 * 8);
}

template <typename T, int NC, bool VEC>
__global__ __launch_bounds__(64 * kFWaves, sizeof(T) == 4 && NC <= 12 ? 2 : 1) void k_forpdn_filter(FFilter a) {
    extern __shared__ unsigned char s_raw[];
    constexpr int VW = 16 / (int)sizeof(T);         // values of a 16-byte LDS access
    constexpr int V = VEC ? VW : 1;                 // values of a global access
    constexpr int LPR = 16 / V, RPS = 64 / LPR, K = 64 / RPS;   // lanes per row, rows per step, steps
    constexpr int P16 = NC * 16, ST = kFStride<T>;
    typedef typename Bands<T, V>::type GT;
    typedef typename Bands<T, VW>::type LT;
    const int p = a.p, G = a.groups;
    T* s_inv = reinterpret_cast<T*>(s_raw);                 // [G][P16]
    T* s_f = s_inv + (size_t)G * P16;                       // [G][P16]
    T* s_all = s_f + (size_t)G * P16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    T* s_row = s_all + (size_t)wave * 64 * ST;              // [64][ST], this wave's
    const int64_t npos = a.npos, ntile = (npos + 63) / 64;
    const HYRES_GLOBAL T* coef = gmem(static_cast<const T*>(a.coef));
    const int lr = lane / LPR, lb = (lane % LPR) * V;       // row and band of a lane's global access
    const int tail = min(16 * (NC - 1) + lb, p - V) - lb;   // last chunk: bands past p read others of the row
    T z[P16];
    uint32_t at[K];                                         // this lane's place in its rows (those past the end: the last)

    // raw values of the tile, in the layout of the global accesses: chunks at constant
    // offsets from the places (an address each would not leave room for the rows)
    auto load = [&](int64_t tile) {
        const int64_t pos0 = tile * 64;
        const int last = npos - pos0 < 64 ? (int)(npos - pos0) - 1 : 63;
        const HYRES_GLOBAL T* src = coef + pos0 * p;
#pragma unroll
        for (int k = 0; k < K; ++k) at[k] = (uint32_t)(min(lr + k * RPS, last) * p + lb);
        static_for<NC>([&](auto cc) {
            constexpr int c = cc;
            static_for<K>([&](auto kc) {
                constexpr int k = kc;
                const GT v = *(const HYRES_GLOBAL GT*)(src + at[k] + (c + 1 < NC ? 16 * c : tail));
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    if constexpr (V == 1) z[16 * c + k] = v;
                    else z[16 * c + k * V + i] = v[i];
                }
            });
        });
    };
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // LDS place of step k of a lane's global layout
    auto turn_place = [&](int k) { return s_row + (lr + k * RPS) * ST + lb; };

    int64_t tile = (int64_t)blockIdx.x * kFWaves + wave;
    if (tile < ntile) load(tile);
    {
        // beta_i = d_i - lam^2 / beta_(i-1), one lane per group; then its quotients
        double* s_beta = reinterpret_cast<double*>(s_all);  // [G][P16]
        if ((int)threadIdx.x < G) {
            const double lam = a.lambda[threadIdx.x];
            double beta = 0.0;
            for (int i = 0; i < p; ++i) {
                const double d = p == 1 ? 1.0 : (i == 0 || i == p - 1) ? 1.0 + lam : 1.0 + 2.0 * lam;
                beta = i == 0 ? d : d - lam * lam / beta;
                s_beta[threadIdx.x * P16 + i] = beta;
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < G * P16; e += 64 * kFWaves) {
            const int j = e / P16, i = e - j * P16;
            const double beta = i < p ? s_beta[e] : 1.0;
            s_inv[e] = i < p ? (T)(1.0 / beta) : (T)0;
            s_f[e] = i < p ? (T)(a.lambda[j] / beta) : (T)0;
        }
        __syncthreads();
    }
    for (; tile < ntile; tile += (int64_t)gridDim.x * kFWaves) {
        const int64_t pos = tile * 64 + lane;
        int j = 0;
        while (j + 1 < G && pos >= a.goff[j + 1]) ++j;
        const T lam = (T)a.lambda[j];
        const T* inv = s_inv + j * P16;
        const T* f = s_f + j * P16;
        T x = 0;
        static_for<NC>([&](auto cc) {
            constexpr int c = cc;
            static_for<K>([&](auto kc) {
                constexpr int k = kc;
#pragma unroll
                for (int i = 0; i < V; ++i) turn_place(k)[i] = z[16 * c + k * V + i];
            });
            wave_sync();
#pragma unroll
            for (int i = 0; i < 16; i += VW) {
                const LT v = *(const LT*)(s_row + lane * ST + i);
                const LT w = *(const LT*)(inv + 16 * c + i);
#pragma unroll
                for (int q = 0; q < VW; ++q) {
                    // bands past p: nothing to carry
                    if (c + 1 < NC || 16 * c + i + q < p) x = (c + i + q == 0 ? v[q] : fma(lam, x, v[q])) * w[q];
                    z[16 * c + i + q] = x;
                }
            }
            wave_sync();
        });
        const int cnt = npos - tile * 64 < 64 ? (int)(npos - tile * 64) : 64;
        HYRES_GLOBAL T* dst = gmem(static_cast<T*>(a.coef)) + tile * 64 * p;
        static_for<NC>([&](auto cc) {
            constexpr int c = NC - 1 - (int)cc;
#pragma unroll
            for (int i = 16 - VW; i >= 0; i -= VW) {
                const LT w = *(const LT*)(f + 16 * c + i);
                LT v;
#pragma unroll
                for (int q = VW - 1; q >= 0; --q) {
                    if (c + 1 == NC && 16 * c + i + q >= p - 1) x = z[16 * c + i + q];
                    else x = fma(w[q], x, z[16 * c + i + q]);
                    v[q] = x;
                }
                *(LT*)(s_row + lane * ST + i) = v;
            }
            wave_sync();
            static_for<K>([&](auto kc) {
                constexpr int k = kc;
                const int r = lr + k * RPS;
                GT v;
#pragma unroll
                for (int i = 0; i < V; ++i) set_band<T, V>(v, i, turn_place(k)[i]);
                if (r < cnt && (c + 1 < NC || 16 * c + lb < p)) *(HYRES_GLOBAL GT*)(dst + at[k] + 16 * c) = v;
            });
            wave_sync();
        });
        if (tile + (int64_t)gridDim.x * kFWaves < ntile) load(tile + (int64_t)gridDim.x * kFWaves);
    }
}

// Bands per thread of a transform level: 16 bytes when both arrays allow it
// (band count and strides whole vectors, aligned), else one.
static bool vec_ok(const void* ptr, int64_t pos, int64_t row, int p, int es) {
    const int V = 16 / es;
    return p % V == 0 && pos % V == 0 && row % V == 0 && reinterpret_cast<uintptr_t>(ptr) % 16 == 0;
}

// Blocks of a transform level: one item of 256 threads each, up to 16 per
// compute unit in turn.
static int level_grid(int64_t nq, int pv, int num_cu) {
    return (int)std::min<int64_t>((nq * pv + 255) / 256, (int64_t)num_cu * 16);
}

hipError_t launch_vdwt_level(int dtype, const VLevel& a, int num_cu, hipStream_t s) {
    const int es = dtype == HYRES_F64 ? 8 : 4;
    const bool vec = vec_ok(a.in, a.ip, a.irow, a.p, es) && vec_ok(a.ll, a.p, a.p, a.p, es) && vec_ok(a.det, a.p, a.p, a.p, es);
    const int grid = level_grid((int64_t)((a.h + 1) / 2) * ((a.w + 1) / 2), vec ? a.p * es / 16 : a.p, num_cu);
    if (dtype == HYRES_F32) {
        if (vec) hipLaunchKernelGGL((k_vdwt_level<float, 4>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_vdwt_level<float, 1>), dim3(grid), dim3(256), 0, s, a);
    } else {
        if (vec) hipLaunchKernelGGL((k_vdwt_level<double, 2>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_vdwt_level<double, 1>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_vidwt_level(int dtype, const VSyn& a, int num_cu, hipStream_t s) {
    const int es = dtype == HYRES_F64 ? 8 : 4;
    const bool vec = vec_ok(a.out, a.op, a.orow, a.p, es) && vec_ok(a.ll, a.p, a.p, a.p, es) && vec_ok(a.det, a.p, a.p, a.p, es);
    const int grid = level_grid((int64_t)a.h * a.w, vec ? a.p * es / 16 : a.p, num_cu);
    if (dtype == HYRES_F32) {
        if (vec) hipLaunchKernelGGL((k_vidwt_level<float, 4>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_vidwt_level<float, 1>), dim3(grid), dim3(256), 0, s, a);
    } else {
        if (vec) hipLaunchKernelGGL((k_vidwt_level<double, 2>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_vidwt_level<double, 1>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_forpdn_lambda(const FLambda& a, int groups, hipStream_t s) {
    hipLaunchKernelGGL(k_forpdn_lambda, dim3(groups), dim3(1024), 0, s, a);
    return hipGetLastError();
}

template <typename T, int NC>
static hipError_t launch_filter_nc(const FFilter& a, int num_cu, hipStream_t s) {
    if (a.p <= 16 * (NC - 1)) {
        if constexpr (NC > 1) return launch_filter_nc<T, NC - 1>(a, num_cu, s);
    }
    const size_t lds = filter_lds((int)sizeof(T), NC, a.groups);
    // blocks that fit a compute unit: the registers hold a row, and LDS
    const int regs = NC * 16 * (int)sizeof(T) / 4 + 56;
    const int per_cu = std::max(1, std::min<int>({512 / regs, (int)((160 * 1024) / lds), 4}));
    const int64_t ntile = (a.npos + 63) / 64;
    const int grid = (int)std::min<int64_t>((ntile + kFWaves - 1) / kFWaves, (int64_t)num_cu * per_cu);
    auto kern = a.p % (16 / (int)sizeof(T)) == 0 ? &k_forpdn_filter<T, NC, true> : &k_forpdn_filter<T, NC, false>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kFWaves), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_forpdn_filter(int dtype, const FFilter& a, int num_cu, hipStream_t s) {
    constexpr int NCM = kMaxBands / 16;
    return dtype == HYRES_F32 ? launch_filter_nc<float, NCM>(a, num_cu, s) : launch_filter_nc<double, NCM>(a, num_cu, s);
}

}  // namespace hyres
