// FP64 small solves of one cube in one workgroup:
//   noise   sigma_i^2 = 1 / (n [G^-1]_ii)           (elimination of the band Gram)
//   whiten  C = D^-1 G D^-1,  D = diag(sigma)
//   eigen   Householder tridiagonalisation of C, eigenvalues by Sturm-count
//           multisection, the top-r eigenvectors of the tridiagonal matrix from a
//           twisted factorisation, modified Gram-Schmidt, back-transformation.
//
// The regression of band i on the other bands leaves the residual sum of
// squares 1/[G^-1]_ii (Schur complement), which is why the noise estimate only
// needs the diagonal of the inverse Gram.
//
// The p x p matrix lives in registers by columns (T tiles of 16 columns, those of
// the largest band count of its class, so that cubes of one class share a launch): lane (g, c) = (lane / 16, lane mod 16) of the wave that owns column
// tile w holds, of column 16 w + c, the rows 4 e + g, e < 4 T.  A vector that
// multiplies the rows is read from LDS as T / 4 registers, lane (g, c) holding its
// entries of rows 4 (16 m + c) + g, and a product with row 4 (16 m + c') + g takes
// the entry of lane c' of the same 16 lanes as its operand (row_newbcast of
// v_fmac_f64): one instruction per entry and no LDS traffic or register for the
// row operand.  Column sums stay in the lane but for two swaps over g, and a
// matrix row, which by symmetry is the next column, leaves the registers with
// one LDS write per wave.  A wave owns one tile up to T = 12 (at most three waves
// and 168 registers per SIMD); beyond, seven waves own two tiles each (two
// waves and 256 registers per SIMD) and keep the rows of the first three tiles,
// dead after 48 steps, in LDS (two tiles per wave from T = 9 on measured 314 us
// against 298 at p = 144).  What bounds it is the chain of a step, about 250
// instructions of one wave at five cycles each beside the products: reductions,
// a square root, a quotient, a barrier.  The previous layout (a thread grid with
// 5 x 9 entries per thread at p = 144, row sums over 16 lanes by DPP, operands of
// both sides from LDS) issued about 480 vector instructions per Householder
// step and wave.  Microseconds before and now at rank 4-10: 32 bands 81, 50; 103
// 375, 200; 128 435, 231; 144 472, 290; 191 867, 428; 224 1490, 706.  Of the 290:
// noise 61, tridiagonalisation 137, Sturm counts 29, twisted factorisation 20,
// back-transformation 36.
#include "hyres_internal.hpp"

namespace hyres {

constexpr int kSmallP = 256;   // LDS vector length (p <= 224)

// Entry of lane C of each row of 16 lanes, to every lane of the row.
template <int C>
__device__ __forceinline__ double row_bcast(double v) {
    long long x = __builtin_bit_cast(long long, v);
    x = __builtin_amdgcn_update_dpp(x, x, 0x150 + C, 0xf, 0xf, true);
    return __builtin_bit_cast(double, x);
}

// Sturm count: number of eigenvalues of the symmetric tridiagonal matrix
// smaller than x, from the sign changes of the leading principal minors
// p_i(x) = (d_i - x) p_{i-1}(x) - e_{i-1}^2 p_{i-2}(x) (a minor that is
// exactly zero counts as positive); both minors are rescaled by a power of two
// every 8 steps so the recursion stays in range.  Lane c of a row of 16 holds
// d_i and e_{i-1}^2 of i = 16 b + c (entries past the matrix: d = 3, e = 0, no sign
// change for x < 3; whole groups of eight of them are left out where the class
// may have them, which those of the class's smallest band count do not pay for); a step is two broadcasts, three FP64 operations and one that
// shifts the sign into a word: 24 issue cycles, no LDS (broadcast 16-byte reads of
// all waves were its bound before, 49 cycles a step).  Call with all sixteen lanes
// of a row active: a lane that is off broadcasts zeros.
template <int T>
__device__ __forceinline__ int sturm_count(const double (&dv)[T], const double (&ev)[T], int p, double x) {
    double pm2 = 0.0, pm1 = 1.0;
    uint32_t bits = 0;                         // signs of the minors, the latest lowest
    int cnt = 0;
    static_for<2 * T>([&](auto h) {
        constexpr int b = decltype(h)::value / 2, c0 = 8 * (decltype(h)::value % 2);
        constexpr int least = 16 * (T <= 2 || (T > 8 && T < 13) ? T - 1 : T - 2);   // bands of the class below
        if (8 * decltype(h)::value > least && 8 * decltype(h)::value >= p) return;
        static_for<8>([&](auto u) {
            constexpr int c = c0 + decltype(u)::value;
            const double pi = fma(row_bcast<c>(dv[b]) - x, pm1, -row_bcast<c>(ev[b]) * pm2);
            bits = __builtin_amdgcn_alignbit(bits, (uint32_t)__double2hiint(pi), 31);
            pm2 = pm1;
            pm1 = pi;
        });
        cnt += __builtin_popcount((bits ^ (bits >> 1)) & 0xffu);
        const int e1 = __builtin_amdgcn_frexp_exp(pm1), e2 = __builtin_amdgcn_frexp_exp(pm2);
        const int e = e1 > e2 ? e1 : e2;
        pm1 = ldexp(pm1, -e);
        pm2 = ldexp(pm2, -e);
    });
    return cnt;
}

// 1 / d and sqrt(s) for normal s > 0: the hardware estimates (24 bits) and
// Newton steps, without the scaling steps of the general division and square
// root (their latency is on the chain of every elimination step).  The last step
// rounds once: against 1 / d and sqrt(s) over 2^20 arguments of every exponent,
// 1 / d differs for 6 of the 256 fractions next to two and nowhere else (by one unit
// in the last place, quotients below 2^-1022 included), the root only below 2^-970
// (by one unit; its residual is subnormal there).
constexpr double kTiny = 0x1p-1022;            // smallest normal number
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    return fma(fma(-d, r, 1.0), r, r);
}
__device__ __forceinline__ double root(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    double w = s * y, h = 0.5 * y;
    const double e = fma(-h, w, 0.5);
    w = fma(w, e, w);
    h = fma(h, e, h);
    return fma(fma(-w, w, s), h, w);
}

// In place: lo = max and hi = min over each aligned group of M lanes (M = 4, 16 or 64).
__device__ __forceinline__ void group_maxmin(double& lo, double& hi, int M) {
    double a;
    a = dpp_f64<0xB1>(lo); lo = a > lo ? a : lo;      // quad_perm [1,0,3,2]
    a = dpp_f64<0xB1>(hi); hi = a < hi ? a : hi;
    a = dpp_f64<0x4E>(lo); lo = a > lo ? a : lo;      // quad_perm [2,3,0,1]
    a = dpp_f64<0x4E>(hi); hi = a < hi ? a : hi;
    if (M == 4) return;
    a = dpp_f64<0x141>(lo); lo = a > lo ? a : lo;     // row_half_mirror
    a = dpp_f64<0x141>(hi); hi = a < hi ? a : hi;
    a = dpp_f64<0x140>(lo); lo = a > lo ? a : lo;     // row_mirror
    a = dpp_f64<0x140>(hi); hi = a < hi ? a : hi;
    if (M == 16) return;
    const double l0 = readlane_f64(lo, 0), l1 = readlane_f64(lo, 16), l2 = readlane_f64(lo, 32),
                 l3 = readlane_f64(lo, 48);
    const double h0 = readlane_f64(hi, 0), h1 = readlane_f64(hi, 16), h2 = readlane_f64(hi, 32),
                 h3 = readlane_f64(hi, 48);
    const double la = l0 > l1 ? l0 : l1, lb = l2 > l3 ? l2 : l3;
    const double ha = h0 < h1 ? h0 : h1, hb = h2 < h3 ? h2 : h3;
    lo = la > lb ? la : lb;
    hi = ha < hb ? ha : hb;
}

// Barrier that orders LDS accesses only: __syncthreads() also waits for the
// global stores in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---- products of register rows with a vector held in lanes (see the top) ----
// a[k] += x[lane C0 + k of this row of 16] * z, k < N.  The wait states at the
// start cover a write of x right before (a DPP operand needs two).
#define HYRES_BC(A, X, Z, C) "v_fmac_f64_dpp " A ", " X ", " Z " row_newbcast:" C " row_mask:0xf bank_mask:0xf\n"
template <int C0, int E0, int N, int E>
__device__ __forceinline__ void axpy_block(double (&a)[E], double x, double z) {
    static_assert(C0 + N <= 16, "within one register of x");
    if constexpr (N == 4) {
        asm("s_nop 1\n" HYRES_BC("%0", "%4", "%5", "%6") HYRES_BC("%1", "%4", "%5", "%7")
                HYRES_BC("%2", "%4", "%5", "%8") HYRES_BC("%3", "%4", "%5", "%9")
            : "+&v"(a[E0]), "+&v"(a[E0 + 1]), "+&v"(a[E0 + 2]), "+&v"(a[E0 + 3])
            : "v"(x), "v"(z), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3));
    } else if constexpr (N == 8) {
        asm("s_nop 1\n" HYRES_BC("%0", "%8", "%9", "%10") HYRES_BC("%1", "%8", "%9", "%11")
                HYRES_BC("%2", "%8", "%9", "%12") HYRES_BC("%3", "%8", "%9", "%13")
                HYRES_BC("%4", "%8", "%9", "%14") HYRES_BC("%5", "%8", "%9", "%15")
                HYRES_BC("%6", "%8", "%9", "%16") HYRES_BC("%7", "%8", "%9", "%17")
            : "+&v"(a[E0]), "+&v"(a[E0 + 1]), "+&v"(a[E0 + 2]), "+&v"(a[E0 + 3]), "+&v"(a[E0 + 4]),
              "+&v"(a[E0 + 5]), "+&v"(a[E0 + 6]), "+&v"(a[E0 + 7])
            : "v"(x), "v"(z), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3), "n"(C0 + 4), "n"(C0 + 5),
              "n"(C0 + 6), "n"(C0 + 7));
    } else {
        static_assert(N == 16, "4, 8 or 16 rows");
        asm("s_nop 1\n" HYRES_BC("%0", "%16", "%17", "0") HYRES_BC("%1", "%16", "%17", "1")
                HYRES_BC("%2", "%16", "%17", "2") HYRES_BC("%3", "%16", "%17", "3")
                HYRES_BC("%4", "%16", "%17", "4") HYRES_BC("%5", "%16", "%17", "5")
                HYRES_BC("%6", "%16", "%17", "6") HYRES_BC("%7", "%16", "%17", "7")
                HYRES_BC("%8", "%16", "%17", "8") HYRES_BC("%9", "%16", "%17", "9")
                HYRES_BC("%10", "%16", "%17", "10") HYRES_BC("%11", "%16", "%17", "11")
                HYRES_BC("%12", "%16", "%17", "12") HYRES_BC("%13", "%16", "%17", "13")
                HYRES_BC("%14", "%16", "%17", "14") HYRES_BC("%15", "%16", "%17", "15")
            : "+&v"(a[E0]), "+&v"(a[E0 + 1]), "+&v"(a[E0 + 2]), "+&v"(a[E0 + 3]), "+&v"(a[E0 + 4]),
              "+&v"(a[E0 + 5]), "+&v"(a[E0 + 6]), "+&v"(a[E0 + 7]), "+&v"(a[E0 + 8]), "+&v"(a[E0 + 9]),
              "+&v"(a[E0 + 10]), "+&v"(a[E0 + 11]), "+&v"(a[E0 + 12]), "+&v"(a[E0 + 13]), "+&v"(a[E0 + 14]),
              "+&v"(a[E0 + 15])
            : "v"(x), "v"(z));
    }
}
// y[k mod 4] += x[lane C0 + k] * a[k], k < N
template <int C0, int E0, int N, int E>
__device__ __forceinline__ void dot_block(const double (&a)[E], double x, double (&y)[4]) {
    if constexpr (N == 4) {
        asm("s_nop 1\n" HYRES_BC("%0", "%4", "%5", "%9") HYRES_BC("%1", "%4", "%6", "%10")
                HYRES_BC("%2", "%4", "%7", "%11") HYRES_BC("%3", "%4", "%8", "%12")
            : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3])
            : "v"(x), "v"(a[E0]), "v"(a[E0 + 1]), "v"(a[E0 + 2]), "v"(a[E0 + 3]), "n"(C0), "n"(C0 + 1),
              "n"(C0 + 2), "n"(C0 + 3));
    } else {
        static_assert(N == 8, "4 or 8 rows");
        asm("s_nop 1\n" HYRES_BC("%0", "%4", "%5", "%13") HYRES_BC("%1", "%4", "%6", "%14")
                HYRES_BC("%2", "%4", "%7", "%15") HYRES_BC("%3", "%4", "%8", "%16")
                HYRES_BC("%0", "%4", "%9", "%17") HYRES_BC("%1", "%4", "%10", "%18")
                HYRES_BC("%2", "%4", "%11", "%19") HYRES_BC("%3", "%4", "%12", "%20")
            : "+&v"(y[0]), "+&v"(y[1]), "+&v"(y[2]), "+&v"(y[3])
            : "v"(x), "v"(a[E0]), "v"(a[E0 + 1]), "v"(a[E0 + 2]), "v"(a[E0 + 3]), "v"(a[E0 + 4]),
              "v"(a[E0 + 5]), "v"(a[E0 + 6]), "v"(a[E0 + 7]), "n"(C0), "n"(C0 + 1), "n"(C0 + 2), "n"(C0 + 3),
              "n"(C0 + 4), "n"(C0 + 5), "n"(C0 + 6), "n"(C0 + 7));
    }
}
#undef HYRES_BC
// All rows from element E0 on.  The first EL elements of a column live in LDS
// (element e at low[e * stride]), the others in a[e - EL].
template <int E0, int EL, int E, int M>
__device__ __forceinline__ void axpy_rows(double (&a)[E - EL], double* low, int stride, const double (&x)[M], double z) {
    if constexpr (E0 < EL) {
        double t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = low[(E0 + k) * stride];
        axpy_block<(E0 & 15), 0, 4>(t, x[E0 >> 4], z);
#pragma unroll
        for (int k = 0; k < 4; ++k) low[(E0 + k) * stride] = t[k];
        __builtin_amdgcn_sched_barrier(0);   // reads hoisted above others would spill
        axpy_rows<E0 + 4, EL, E, M>(a, low, stride, x, z);
    } else if constexpr (E0 < E) {
        constexpr int room = 16 - (E0 & 15), len = room < E - E0 ? room : E - E0;
        constexpr int N = len >= 16 ? 16 : len >= 8 ? 8 : 4;
        axpy_block<(E0 & 15), E0 - EL, N>(a, x[E0 >> 4], z);
        axpy_rows<E0 + N, EL, E, M>(a, low, stride, x, z);
    }
}
template <int E0, int EL, int E, int M>
__device__ __forceinline__ void dot_rows(const double (&a)[E - EL], const double* low, int stride, const double (&x)[M],
                                         double (&y)[4]) {
    if constexpr (E0 < EL) {
        double t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = low[(E0 + k) * stride];
        dot_block<(E0 & 15), 0, 4>(t, x[E0 >> 4], y);
        __builtin_amdgcn_sched_barrier(0);
        dot_rows<E0 + 4, EL, E, M>(a, low, stride, x, y);
    } else if constexpr (E0 < E) {
        constexpr int room = 16 - (E0 & 15), len = room < E - E0 ? room : E - E0;
        constexpr int N = len >= 8 ? 8 : 4;
        dot_block<(E0 & 15), E0 - EL, N>(a, x[E0 >> 4], y);
        dot_rows<E0 + N, EL, E, M>(a, low, stride, x, y);
    }
}

// Sum over the four rows of 16 lanes (g), to every lane: the B operand of the
// 4 x 4 x 4 product of four blocks holds row k = g of column c in lane (g, c), so
// a product with ones is the sum, one instruction of 28 cycles.
__device__ __forceinline__ double rows_sum(double v) { return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0); }
// Sum over the wave, to every lane: as the A operand the row sums come out
// transposed within each block of four columns; their sum over g is the block's,
// and two mirrors within the 16 lanes add the blocks.
__device__ __forceinline__ double wave_total(double v) {
    v = rows_sum(__builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0));
    v += dpp_f64<0x141>(v);   // row_half_mirror
    v += dpp_f64<0x140>(v);   // row_mirror
    return v;
}

// Element E0 + q of a column for the wave-uniform q < N (every index a constant:
// the array stays in registers).
template <int E0, int N, int EL, int E>
__device__ __forceinline__ double pick(const double (&a)[E - EL], const double* low, int stride, int q) {
    if constexpr (N > 1 && E0 + N > E) {
        return pick<E0, N - 1, EL, E>(a, low, stride, q);
    } else if constexpr (E0 + N <= EL) {
        return low[(E0 + q) * stride];
    } else if constexpr (N == 1) {
        return a[E0 - EL];
    } else {
        const double v = pick<E0, N - 1, EL, E>(a, low, stride, q);
        return q == N - 1 ? a[E0 + N - 1 - EL] : v;
    }
}

// Shape of the column layout of T tiles.
template <int T>
struct Cols {
    static constexpr int NC = T >= 13 ? 2 : 1;           // column tiles per wave
    static constexpr int W = (T + NC - 1) / NC;          // waves that own columns
    static constexpr int NW = W > 8 ? W : T >= 5 ? 8 : 4;  // waves of the block
    static constexpr int E = 4 * T;                      // rows per lane
    static constexpr int EL = NC == 2 ? E - 44 : 0;      // ... of which in LDS: registers hold 2 x 44 rows
    static constexpr int M = (T + 3) / 4;                // registers of a row vector
    static constexpr int SP = M % 2 ? 16 * M : 16 * M + 16;   // LDS stride of its four parts: 16 mod 32 doubles
    static constexpr int Q = (T + 3) / 4;                // 64-entry pieces of a vector
    static constexpr int PL = 64 * Q;
};
// LDS position of row (or, by symmetry, column) i of a row vector
template <int T>
__device__ __forceinline__ int slot_of(int i) { return (i & 3) * Cols<T>::SP + (i >> 2); }

template <int T>
__global__ __launch_bounds__(64 * Cols<T>::NW) void k_small(const CubeDesc* __restrict__ descs,
                                                            const int* __restrict__ cubes, int ncls) {
    typedef Cols<T> CL;
    constexpr int NW = CL::NW, NTH = 64 * NW, NC = CL::NC, W = CL::W, E = CL::E, EL = CL::EL, M = CL::M,
                  SP = CL::SP;
    constexpr int Q = CL::Q, PL = CL::PL;
    constexpr int VPW = (kMaxRank + NW - 1) / NW;   // eigenvectors per wave
    if ((int)blockIdx.x >= ncls) return;
    const CubeDesc& d = descs[cubes[blockIdx.x]];
    const int p = d.p, r = d.r;
    const double nn = (double)d.n;
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    __shared__ double s_row[2][2][4 * SP];           // matrix rows (noise: pairs), u and the next row (eigen)
    __shared__ double s_u[4 * SP];
    __shared__ double s_col[2][PL];
    __shared__ double s_sig[PL];
    __shared__ double s_dd[PL], s_ee[PL], s_hb[PL], s_ev[PL];
    // the LDS rows of the columns, then multipliers of the top-down and of the
    // bottom-up factorisation [i][g], and the eigenvectors of the tridiagonal / of C
    constexpr int kPool = NC * EL * 64 * W > 3 * PL * kMaxRank ? NC * EL * 64 * W : 3 * PL * kMaxRank;
    __shared__ double s_pool[kPool];
    double* const s_zL = s_pool;
    double* const s_zU = s_pool + PL * kMaxRank;
    double (*const s_z)[PL] = reinterpret_cast<double (*)[PL]>(s_pool + 2 * PL * kMaxRank);
    __shared__ double s_red[4];
    __shared__ int s_kb[kMaxRank];                   // twist indices
    __shared__ double s_cross[kMaxRank][kMaxRank + 1];   // rank by SURE: sum_{j>=k} l_i / (l_i - l_j), [i][k]
    __shared__ int s_rank;                           // rank used
    __shared__ double s_chk[3][NW];                  // eigenpair check: residual, norm of C, orthonormality
    __shared__ int s_flags;

    if (t == 0) s_flags = 0;
    for (int i = t; i < 4 * SP; i += NTH) {          // the padding of the row vectors stays zero
        s_row[0][0][i] = s_row[0][1][i] = s_row[1][0][i] = s_row[1][1][i] = 0.0;
        s_u[i] = 0.0;
    }
    int flags = 0;
    HYRES_STAMP(d, 0);
    double A[NC][E - EL];
    constexpr int LS = NC * 64 * W;                  // stride of the LDS rows
    double* low[NC];
    // column and slot of this lane per column tile (tiles beyond T: column -1)
    int col[NC], own[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int tile = wave + W * j;
        col[j] = wave < W && tile < T ? 16 * tile + c : -1;
        own[j] = col[j] >= 0 ? slot_of<T>(col[j]) : 0;
        low[j] = s_pool + (j * W + (wave < W ? wave : 0)) * 64 + lane;
    }
    const HYRES_GLOBAL double* G = gmem(static_cast<const double*>(d.G));
    HYRES_GLOBAL double* hv = gmem(d.hv);
    int clampc[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) clampc[j] = min(max(col[j], 0), p - 1);
    // this lane's columns of G, every load in flight at once (entries beyond p
    // read the last row or column and are replaced by the caller)
    auto load_columns = [&]() {
        static_for<NC * E>([&](auto x) {
            constexpr int j = decltype(x)::value / E, e = decltype(x)::value % E;
            const double v = G[(uint32_t)(min(4 * e + g, p - 1) * p + clampc[j])];
            if constexpr (e < EL) low[j][e * LS] = v;
            else A[j][e - EL] = v;
        });
    };
    __syncthreads();

    // ---------------------------------------------------------------- noise
    // Elimination L D L^T of G without pivoting, building L^-1 in place: after the
    // pivot k column k of the matrix holds column k of L^-1 times d_k below the
    // diagonal, and [G^-1]_ii = sum_k (L^-1)_ki^2 / d_k is summed as the rows are
    // finished.  One update serves every column n, A_in -= x_i c_n with x the pivot
    // column: c_n = row_n / d_k, and 2 for n = k (x - 2 x = -x is exact).  Rows up to
    // the pivot are dead; what the update leaves there is never read.  Pivots in
    // pairs, one barrier each: row k1 after the k0 step is formed by every lane.
    if (d.mode & 1) {
        if (wave < W) {
            load_columns();
            static_for<NC * E>([&](auto x) {
                constexpr int j = decltype(x)::value / E, e = decltype(x)::value % E;
                const int i = 4 * e + g, n = col[j];
                double v;
                if constexpr (e < EL) v = low[j][e * LS];
                else v = A[j][e - EL];
                v = i < p && n >= 0 && n < p ? v : (i == n ? 1.0 : 0.0);
                if constexpr (e < EL) low[j][e * LS] = v;
                else A[j][e - EL] = v;
            });
        }
        // diagonal of G for the pivot test (s_ev is free until the eigenvalues)
        for (int i = t; i < PL; i += NTH) s_ev[i] = i < p ? d.G[(int64_t)i * p + i] : 1.0;
        double acc[NC], dself[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            acc[j] = 0.0;
            dself[j] = 1.0;
        }
        static_for<T>([&](auto tc) {
            constexpr int t0 = decltype(tc)::value, m0 = t0 / 4;
#pragma unroll 1
            for (int kk = 0; kk < 16; kk += 2) {   // unrolled, its code would not fit the instruction cache
                const int k0 = 16 * t0 + kk, k1 = k0 + 1;
                if (k0 >= p) break;
                double (*row)[4 * SP] = s_row[(kk >> 1) & 1];
                const int gr = g - (kk & 3);             // 0: holds row k0, 1: row k1
                if (wave < W) {
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const double v = pick<4 * t0, 4, EL, E>(A[j], low[j], LS, kk >> 2);
                        if (col[j] >= 0 && (gr == 0 || gr == 1)) row[gr][own[j]] = v;
                    });
                }
                __syncthreads();
                // the pivot is the regression residual of band k on the bands before it
                double d0 = row[0][slot_of<T>(k0)];
                const double r01 = row[0][slot_of<T>(k1)], r11 = row[1][slot_of<T>(k1)];
                if (!(d0 > 1e-12 * s_ev[k0])) {
                    flags |= HYRES_DEV_NOT_PD;
                    d0 = 1.0;
                }
                const double inv0 = recip(d0), m01 = r01 * inv0;
                double d1 = fma(-r01, m01, r11);
                if (!(d1 > 1e-12 * s_ev[k1])) {
                    flags |= HYRES_DEV_NOT_PD;
                    d1 = 1.0;
                }
                const double inv1 = recip(d1);
                if (wave < W) {
                    double x0[M], x1[M];
#pragma unroll
                    for (int m = m0; m < M; ++m) {
                        x0[m] = row[0][g * SP + 16 * m + c];
                        x1[m] = fma(-m01, x0[m], row[1][g * SP + 16 * m + c]);
                    }
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const int n = col[j];
                        const double r0 = row[0][own[j]];
                        const double c0 = n == k0 ? 2.0 : r0 * inv0;
                        const double r1 = fma(-r01, c0, row[1][own[j]]);
                        const double c1 = n == k1 ? 2.0 : r1 * inv1;
                        if (n < k0) acc[j] = fma(r0, c0, acc[j]);
                        if (n == k0) dself[j] = d0;
                        if (n < k1) acc[j] = fma(r1, c1, acc[j]);
                        if (n == k1) dself[j] = d1;
                        axpy_rows<4 * t0, EL, E, M>(A[j], low[j], LS, x0, -c0);
                        axpy_rows<4 * t0, EL, E, M>(A[j], low[j], LS, x1, -c1);
                    });
                }
            }
        });
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int n = col[j];
            if (g == 0 && n >= 0 && n < p) {
                const double inv = 1.0 / dself[j], gii = fma(acc[j] * inv, inv, inv);
                double s = 1.0;
                if (gii > 0.0 && !(flags & HYRES_DEV_NOT_PD)) s = sqrt(1.0 / (nn * gii));
                else flags |= HYRES_DEV_NOT_PD;
                s_sig[n] = s;
                d.sigma[n] = s;
            }
        }
    } else if (t < p) {
        const double s = d.sigma_in ? d.sigma_in[t] : 1.0;
        s_sig[t] = s;
        d.sigma[t] = s;
    }
    __syncthreads();

    HYRES_STAMP(d, 1);
    if (d.mode & 2) {
        // ------------------------------------------------------- whitened Gram
        if (wave < W) {
            double sn[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) sn[j] = s_sig[clampc[j]];
            load_columns();
            static_for<NC * E>([&](auto x) {
                constexpr int j = decltype(x)::value / E, e = decltype(x)::value % E;
                const int i = 4 * e + g, n = col[j];
                double v;
                if constexpr (e < EL) v = low[j][e * LS];
                else v = A[j][e - EL];
                v = i < p && n >= 0 && n < p ? v / (s_sig[i] * sn[j]) : 0.0;
                if constexpr (e < EL) low[j][e * LS] = v;
                else A[j][e - EL] = v;
            });
        }
        __syncthreads();

        // ------------------------------------------------ tridiagonalisation
        // Step k, x the entries of row k beyond the diagonal: v = x - alpha e_{k+1},
        // u = beta A v, A <- A - v w^T - w v^T with w = u - K v, K = (beta / 2) u^T v, that
        // is A_in -= v_i (u_n - 2 K v_n) + u_i v_n.  A v = A x - alpha A e_{k+1}: the
        // products with x do not wait for the norm that gives alpha.  One barrier a
        // step: the waves publish A v and row k + 1 before the update, and every wave
        // forms the next x from them (in row layout, and for its own columns).
        double xr[M], xo[NC];
        static_for<NC>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            const double v = pick<0, 1, EL, E>(A[j], low[j], LS, 0);
            if (col[j] >= 0 && g == 0) {
                s_u[own[j]] = col[j] > 0 ? v : 0.0;
                if (col[j] == 0) s_dd[0] = v;
            }
        });
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; ++m) xr[m] = s_u[g * SP + 16 * m + c];
#pragma unroll
        for (int j = 0; j < NC; ++j) xo[j] = s_u[own[j]];
        static_for<T>([&](auto tc) {
            constexpr int t0 = decltype(tc)::value, m0 = t0 / 4, mn = (t0 + 1) / 4 < M ? (t0 + 1) / 4 : m0;
#pragma unroll 1
            for (int kk = 0; kk < 16; ++kk) {
                const int k = 16 * t0 + kk;
                if (k >= p - 2) break;
                double* su = s_row[k & 1][0];
                double* sa = s_row[k & 1][1];
                bool act[NC], any = false;
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const int tile = wave + W * j;
                    act[j] = wave < W && tile < T && tile >= t0;
                    any |= act[j];
                }
                double y[NC], v[NC], v1 = 0.0, alpha = 0.0, beta = 0.0;
                if (any) {
                    double ss = 0.0;
#pragma unroll
                    for (int m = m0; m < M; ++m) ss = fma(xr[m], xr[m], ss);
                    ss = wave_total(ss);
                    // entry k + 1 of x, in the lane and register of its row
                    const int l1 = ((k + 1) & 3) * 16 + (((k + 1) >> 2) & 15);
                    const double x1 = readlane_f64(kk == 15 ? xr[mn] : xr[m0], l1);
                    double a1[NC];
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        y[j] = a1[j] = 0.0;
                        if (act[j]) {
                            a1[j] = pick<4 * t0, 5, EL, E>(A[j], low[j], LS, (kk + 1) >> 2);
                            double q[4] = {0.0, 0.0, 0.0, 0.0};
                            dot_rows<4 * t0, EL, E, M>(A[j], low[j], LS, xr, q);
                            y[j] = (q[0] + q[1]) + (q[2] + q[3]);
                        }
                    });
                    // a row whose squares vanish is taken as tridiagonal already
                    const bool some = ss >= kTiny;
                    const double nr = root(fmax(ss, kTiny)), nrm = some ? nr : 0.0;
                    alpha = x1 >= 0.0 ? -nrm : nrm;
                    const double b = recip(nr * (nr + fabs(x1)));     // 2 / v^T v
                    beta = some ? b : 0.0;
                    v1 = x1 - alpha;
                    const bool row1 = g == ((kk + 1) & 3);
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        v[j] = 0.0;
                        if (act[j]) {
                            y[j] = rows_sum(row1 ? fma(-alpha, a1[j], y[j]) : y[j]);
                            v[j] = col[j] == k + 1 ? v1 : xo[j];
                            if (row1) {
                                su[own[j]] = y[j];
                                sa[own[j]] = a1[j];
                            }
                        }
                    });
                    if (kk == 15) xr[mn] = lane == l1 ? v1 : xr[mn];      // v in place of x
                    else xr[m0] = lane == l1 ? v1 : xr[m0];
                }
                lds_barrier();
                if (any) {
                    double yr[M], xn[M], q = 0.0;        // A v and row k + 1 in row layout
                    const double y1 = su[slot_of<T>(k + 1)];
#pragma unroll
                    for (int m = m0; m < M; ++m) {
                        yr[m] = su[g * SP + 16 * m + c];
                        xn[m] = sa[g * SP + 16 * m + c];
                    }
#pragma unroll
                    for (int m = m0; m < M; ++m) {
                        // rows up to k hold what their waves left there
                        yr[m] = beta * yr[m];
                        q = fma(xr[m], yr[m], q);
                    }
                    q = wave_total(q);                   // beta v^T A v
                    const double u1 = beta * y1;
                    double u[NC];
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (act[j]) {
                            u[j] = beta * y[j];
                            if (g == 1 && col[j] < p) hv[(uint32_t)(k * p + col[j])] = v[j];
                            axpy_rows<4 * t0, EL, E, M>(A[j], low[j], LS, yr, -v[j]);
                        }
                    });
                    if (lane == 0) {
                        s_ee[k] = alpha;                 // the same value from every wave
                        s_hb[k] = beta;
                    }
                    const double K2 = beta * q;
                    // row k + 1 after the update
#pragma unroll
                    for (int m = m0; m < M; ++m) {
                        const int i = 4 * (16 * m + c) + g;
                        const double nx = fma(-u1, xr[m], fma(-v1, fma(-K2, xr[m], yr[m]), xn[m]));
                        xn[m] = i > k + 1 ? nx : 0.0;
                    }
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (act[j]) {
                            const double z = fma(-K2, v[j], u[j]);
                            const double nx = fma(-u1, v[j], fma(-v1, z, sa[own[j]]));
                            if (col[j] == k + 1) s_dd[k + 1] = nx;
                            xo[j] = col[j] > k + 1 ? nx : 0.0;
                            axpy_rows<4 * t0, EL, E, M>(A[j], low[j], LS, xr, -z);
                        }
                    });
#pragma unroll
                    for (int m = m0; m < M; ++m) xr[m] = xn[m];
                }
            }
        });
        __syncthreads();
        constexpr int EE = E > 8 ? 8 : E;                // rows of the last two tiles
        static_for<NC * EE>([&](auto x) {
            constexpr int j = decltype(x)::value / EE, e = E - EE + decltype(x)::value % EE;
            const int i = 4 * e + g, n = col[j];
            if (i == n && i >= p - 2 && i < p) s_dd[i] = A[j][e - EL];
            if (i == p - 1 && n == p - 2) s_ee[p - 2] = A[j][e - EL];
        });
        __syncthreads();

        HYRES_STAMP(d, 2);
        // ------------------------------------------------ eigenvalues (all)
        if (wave == 0) {
            double m = 0.0;
            for (int i = lane; i < p; i += 64) {
                double rr = fabs(s_dd[i]);
                if (i > 0) rr += fabs(s_ee[i - 1]);
                if (i < p - 1) rr += fabs(s_ee[i]);
                m = rr > m ? rr : m;
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                const double q = __shfl_xor(m, o, 64);
                m = q > m ? q : m;
            }
            if (lane == 0) s_red[0] = m > 0.0 ? m : 1.0;
        }
        __syncthreads();
        const double gmax = s_red[0];
        const double sc = 1.0 / gmax;
        double dv[T], ev2[T];                            // scaled d_i and e_{i-1}^2 of i = 16 b + c
#pragma unroll
        for (int b = 0; b < T; ++b) {
            const int i = 16 * b + c;
            const double es = i > 0 && i < p ? s_ee[i - 1] * sc : 0.0;
            dv[b] = i < p ? s_dd[i] * sc : 3.0;
            ev2[b] = es * es;
        }
        // Multisection: M lanes per eigenvalue evaluate the Sturm count at M
        // interior points, shrinking the bracket M+1 times per iteration.
        // Only the top r+1 eigenvalues are needed by the solve; all p are
        // computed when requested.
        {
            const int nev = (d.mode & 16) ? p : (r + 1 < p ? r + 1 : p);
            // one wave per SIMD counts as fast as one wave alone
            const int M = nev * 64 <= 256 ? 64 : (nev * 16 <= 2 * NTH ? 16 : 4);
            const int iters = M == 64 ? 9 : (M == 16 ? 14 : 24);
            const double inv_m1 = 1.0 / (double)(M + 1);
            const int m = t % M;
            const int nslot = NTH / M;
            for (int g0 = 0; g0 < nev; g0 += nslot) {
                // whole rows of 16 lanes: a group of a row beyond the last eigenvalue
                // counts along on the last one
                if (g0 + (t & ~15) / M < nev) {
                    const int slot = g0 + t / M, g = min(slot, nev - 1);
                    const int midx = p - 1 - g;        // ascending index of the g-th largest
                    double lo = -1.0 - 1e-12, hi = 1.0 + 1e-12;
                    for (int it = 0; it < iters; ++it) {
                        const double x = lo + (hi - lo) * ((double)(m + 1) * inv_m1);
                        const int cnt = sturm_count<T>(dv, ev2, p, x);
                        const bool below = cnt <= midx;   // x <= lambda
                        double lo_c = below ? x : lo;
                        double hi_c = below ? hi : x;
                        // largest lower and smallest upper end over the M lanes of
                        // the group: quads and rows by DPP, whole waves by readlane
                        group_maxmin(lo_c, hi_c, M);
                        lo = lo_c;
                        hi = hi_c;
                    }
                    if (m == 0 && slot < nev) {
                        const double ev = 0.5 * (lo + hi) * gmax;
                        s_ev[g] = ev;
                        if (d.evals) d.evals[g] = ev;
                    }
                }
            }
        }
        __syncthreads();

        // ----------------------------------------------- data-chosen rank
        // (eigenvalues in s_ev, descending).  HySime on the whitened cube:
        // every eigenvalue above twice the noise power n.  SURE: the rank k
        // minimising sum_{j>=k} lambda_j - n p + 2 df(k) (0-based j), df(k) =
        // k (n - p + 1) + k (k - 1) + 2 sum_{i<k<=j} lambda_i / (lambda_i -
        // lambda_j), every eigenvalue known; the cross sums are spread over
        // the threads, one (i, k) pair each.
        if (t == 0) s_rank = r;
        if (d.mode & kModeRankSure) {
            for (int e = t; e < r * r; e += NTH) {
                const int i = e / r, k = e % r + 1;
                double acc = 0.0;
                if (i < k) {
                    const double li = s_ev[i];
                    for (int j = k; j < p; ++j) acc += li / (li - s_ev[j]);
                }
                s_cross[i][k] = acc;
            }
            __syncthreads();
            if (t == 0) {
                const double n = (double)d.n, pp = (double)p;
                double tail = 0.0;                       // sum_{j >= k} lambda_j
                for (int j = r; j < p; ++j) tail += s_ev[j];
                double best = __builtin_inf();
                int bk = 1;
                for (int k = r; k >= 1; --k) {
                    double cr = 0.0;
                    for (int i = 0; i < k; ++i) cr += s_cross[i][k];
                    const double df = k * (n - pp + 1.0) + k * (k - 1.0) + 2.0 * cr;
                    const double sv = tail - n * pp + 2.0 * df;
                    if (sv <= best) {     // descending k: the last minimum is the smallest rank
                        best = sv;
                        bk = k;
                    }
                    tail += s_ev[k - 1];
                }
                s_rank = bk;
            }
        } else if ((d.mode & kModeRankHySime) && t == 0) {
            const double thr = 2.0 * (double)d.n;
            int k = 0;
            while (k < r && s_ev[k] > thr) ++k;
            s_rank = k < 1 ? 1 : k;
        }
        __syncthreads();
        const int kr = s_rank;

        HYRES_STAMP(d, 3);
        // ---------------------------- eigenvectors of the tridiagonal matrix
        // Twisted factorisation at each eigenvalue mu: the top-down pivots D_i
        // (wave 0) and the bottom-up pivots R_i with multipliers U_i (wave 1)
        // run at the same time; the twist index minimises |D_i + R_i - (d_i - mu)|
        // (largest index on ties); then the two halves of the vector are
        // solved from the twist outwards, again on two waves.
        const double pivmin = gmax * 1e-290;
        if (wave == 0 && lane < r) {
            const int g = lane;
            const double mu = s_ev[g];
            double D = s_dd[0] - mu;
#pragma unroll 4
            for (int i = 0; i < p - 1; ++i) {
                if (fabs(D) < pivmin) D = D < 0.0 ? -pivmin : pivmin;
                const double e = s_ee[i], l = e / D;
                s_zL[i * kMaxRank + g] = l;
                D = (s_dd[i + 1] - mu) - e * l;
            }
        } else if (wave == 1 && lane < r) {
            const int g = lane;
            const double mu = s_ev[g];
            double R = s_dd[p - 1] - mu;
            if (fabs(R) < pivmin) R = R < 0.0 ? -pivmin : pivmin;
            s_z[g][p - 1] = R;
#pragma unroll 4
            for (int i = p - 2; i >= 0; --i) {
                const double e = s_ee[i];
                const double U = e / R;
                s_zU[i * kMaxRank + g] = U;
                R = (s_dd[i] - mu) - U * e;
                if (fabs(R) < pivmin) R = R < 0.0 ? -pivmin : pivmin;
                s_z[g][i] = R;
            }
        }
        __syncthreads();
        // twist index of vector g = wave + NW v: argmin over the lanes of the wave
        int kb_w[VPW];
#pragma unroll
        for (int v = 0; v < VPW; ++v) {
            const int g = wave + NW * v;
            kb_w[v] = 0;
            if (g < r) {
                double best = __builtin_inf();
                int bi = -1;
                for (int i = lane; i < p; i += 64) {
                    // D_i - (d_i - mu) is minus the multiplier above times its off-diagonal
                    const double gam = fabs(s_z[g][i] - (i > 0 ? s_ee[i - 1] * s_zL[(i - 1) * kMaxRank + g] : 0.0));
                    if (gam <= best) {           // ascending i: the last minimum is the largest index
                        best = gam;
                        bi = i;
                    }
                }
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) {
                    const double ob = __shfl_xor(best, o, 64);
                    const int oi = __shfl_xor(bi, o, 64);
                    if (ob < best || (ob == best && oi > bi)) {
                        best = ob;
                        bi = oi;
                    }
                }
                kb_w[v] = bi;
            }
        }
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int v = 0; v < VPW; ++v) {
                const int g = wave + NW * v;
                if (g < r) s_kb[g] = kb_w[v];
            }
        }
        __syncthreads();
        if (wave == 0 && lane < r) {
            const int g = lane, kb = s_kb[g];
            double z = 1.0;
            s_z[g][kb] = 1.0;
#pragma unroll 4
            for (int i = kb - 1; i >= 0; --i) {
                z = -s_zL[i * kMaxRank + g] * z;
                s_z[g][i] = z;
            }
        } else if (wave == 1 && lane < r) {
            const int g = lane, kb = s_kb[g];
            double z = 1.0;
#pragma unroll 4
            for (int i = kb; i < p - 1; ++i) {
                z = -s_zU[i * kMaxRank + g] * z;
                s_z[g][i + 1] = z;
            }
        }
        __syncthreads();

        HYRES_STAMP(d, 4);
        // ---- modified Gram-Schmidt; vector g = wave + NW*v stays in registers of its wave
        double zr[VPW][Q];
#pragma unroll
        for (int v = 0; v < VPW; ++v) {
            const int g = wave + NW * v;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int i = lane + 64 * q;
                zr[v][q] = (g < r && i < p) ? s_z[g][i] : 0.0;
            }
        }
        __syncthreads();
        for (int i = 0; i < r; ++i) {
            double* shared_zi = s_col[i & 1];
            if (wave == i % NW) {
#pragma unroll
                for (int v = 0; v < VPW; ++v) {
                    if (v == i / NW) {
                        double s = 0.0;
#pragma unroll
                        for (int q = 0; q < Q; ++q) s = fma(zr[v][q], zr[v][q], s);
                        s = wave_sum(s);
                        const double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
#pragma unroll
                        for (int q = 0; q < Q; ++q) {
                            zr[v][q] *= inv;
                            shared_zi[lane + 64 * q] = zr[v][q];
                        }
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < VPW; ++v) {
                const int g = wave + NW * v;
                if (g > i && g < r) {
                    double s = 0.0;
#pragma unroll
                    for (int q = 0; q < Q; ++q) s = fma(shared_zi[lane + 64 * q], zr[v][q], s);
                    s = wave_sum(s);
#pragma unroll
                    for (int q = 0; q < Q; ++q) zr[v][q] = fma(-s, shared_zi[lane + 64 * q], zr[v][q]);
                }
            }
        }

        HYRES_STAMP(d, 5);
        // -------------------------- back-transformation v = H_0 ... H_{p-3} z
        // On the FP64 matrix cores, sixteen reflectors at a time: a wave holds the
        // rows of one or two tiles of the vectors as accumulators (16 rows x 16
        // vectors, which is also the B operand of a product over those rows).
        // With S = H z and the products H H^T of the sixteen (summed over the
        // waves through LDS), the j-th of them multiplies its reflector by
        // t_j = hb_j (S_j - sum_{i<j} (h_j^T h_i) t_i), a substitution that every wave
        // does for itself, and z -= H^T t.  One at a time, a wave sum on the chain of
        // each reflector, it took 31 us at p = 144.
        {
            constexpr int TPW = (T + NW - 1) / NW;
            constexpr int NP = T < NW ? T : NW;          // waves that hold tiles
            double* part = s_pool;                       // [wave][S, H H^T][element][lane]
            static_assert(NP * 512 <= 2 * PL * kMaxRank, "below the vectors");
#pragma unroll
            for (int v = 0; v < VPW; ++v) {
                const int gv = wave + NW * v;
                if (gv < r) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) s_z[gv][lane + 64 * q] = zr[v][q];
                }
            }
            __syncthreads();
            v4d Z[TPW];
            double ha[TPW][4], ht[TPW][4], na[TPW][4], nt[TPW][4];
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * (wave + NW * q) + g + 4 * v;
                    Z[q][v] = c < r && i < p ? s_z[c < r ? c : 0][i < p ? i : 0] : 0.0;
                }
            // reflectors k1, k1 - 1, ... k1 - 15 on this wave's rows, by (reflector
            // lane, row) and by (row lane, reflector); entries outside the reflector
            // are read at 0 and cleared at their use, a group later
            auto inside = [&](int k, int i) { return k >= 0 && i > k && i < p; };
            auto entry = [&](int k, int i) { return hv[inside(k, i) ? (uint32_t)(k * p + i) : 0u]; };
            auto fetch = [&](int k1, double (&a)[TPW][4], double (&h)[TPW][4]) {
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i0 = 16 * (wave + NW * q);
                        a[q][e] = entry(k1 - c, i0 + 4 * e + g);
                        h[q][e] = entry(k1 - 4 * e - g, i0 + c);
                    }
            };
            if (p >= 3) fetch(p - 3, ha, ht);
#pragma unroll 1
            for (int k1 = p - 3; k1 >= 0; k1 -= 16) {
                if (k1 >= 16) fetch(k1 - 16, na, nt);
                v4d S = {0.0, 0.0, 0.0, 0.0}, R = S;
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double h = inside(k1 - c, 16 * (wave + NW * q) + 4 * e + g) ? ha[q][e] : 0.0;
                        S = mfma4d(h, Z[q][e], S);
                        R = mfma4d(h, h, R);
                    }
                if (wave < NP) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        part[wave * 512 + e * 64 + lane] = S[e];
                        part[wave * 512 + 256 + e * 64 + lane] = R[e];
                    }
                }
                lds_barrier();
                for (int e = t; e < 512; e += NTH) {
                    double x = 0.0;
#pragma unroll
                    for (int w = 0; w < NP; ++w) x += part[w * 512 + e];
                    part[e] = x;
                }
                lds_barrier();
                double acc[16], tb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[j] = part[16 * j + c];
                static_for<16>([&](auto ic) {
                    constexpr int i = decltype(ic)::value, b0 = (i + 1) / 4 * 4;
                    const double hb = k1 - i >= 0 ? s_hb[k1 - i < 0 ? 0 : k1 - i] : 0.0;
                    const double ti = -hb * acc[i];
                    const double row = part[256 + 16 * i + c];
                    if constexpr (16 - b0 == 16) axpy_block<0, 0, 16>(acc, row, ti);
                    if constexpr (16 - b0 == 12) axpy_block<4, 4, 4>(acc, row, ti);
                    if constexpr (16 - b0 == 12 || 16 - b0 == 8) axpy_block<8, 8, 8>(acc, row, ti);
                    if constexpr (16 - b0 == 4) axpy_block<12, 12, 4>(acc, row, ti);
                    tb[i / 4] = g == i % 4 ? ti : tb[i / 4];
                });
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool in = inside(k1 - 4 * e - g, 16 * (wave + NW * q) + c);
                        Z[q] = mfma4d(in ? ht[q][e] : 0.0, tb[e], Z[q]);
                        ha[q][e] = na[q][e];
                    }
#pragma unroll
                for (int q = 0; q < TPW; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) ht[q][e] = nt[q][e];
                lds_barrier();
            }
#pragma unroll
            for (int q = 0; q < TPW; ++q)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = 16 * (wave + NW * q) + g + 4 * v;
                    if (c < r && i < p) s_z[c][i] = Z[q][v];
                }
            __syncthreads();
#pragma unroll
            for (int v = 0; v < VPW; ++v) {
                const int gv = wave + NW * v;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int i = lane + 64 * q;
                    zr[v][q] = gv < r && i < p ? s_z[gv][i] : 0.0;
                }
            }
        }
        HYRES_STAMP(d, 6);
        if (wave < r) {
            // sign rule: the entry of largest magnitude is positive (lowest index on ties)
#pragma unroll
            for (int v = 0; v < VPW; ++v) {
                const int g = wave + NW * v;
                if (g < r) {
                    double bv = -1.0, bs = 1.0;
                    int bi = 0x7fffffff;
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const int i = lane + 64 * q;
                        if (i < p && fabs(zr[v][q]) > bv) {
                            bv = fabs(zr[v][q]);
                            bi = i;
                            bs = zr[v][q];
                        }
                    }
#pragma unroll
                    for (int o = 32; o >= 1; o >>= 1) {
                        const double ov = __shfl_xor(bv, o, 64);
                        const int oi = __shfl_xor(bi, o, 64);
                        const double os = __shfl_xor(bs, o, 64);
                        if (ov > bv || (ov == bv && oi < bi)) {
                            bv = ov;
                            bi = oi;
                            bs = os;
                        }
                    }
                    const double sgn = bs < 0.0 ? -1.0 : 1.0;
                    int bad = 0;
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        const int i = lane + 64 * q;
                        if (i < p) {
                            // components beyond the chosen rank are zero
                            const double val = g < kr ? zr[v][q] * sgn : 0.0;
                            bad |= !__builtin_isfinite(val);
                            s_z[g][i] = val;
                            d.V[(int64_t)g * p + i] = val;
                        }
                    }
                    if (__any(bad)) flags |= HYRES_DEV_EIGH_NOCONV;
                }
            }
        }
        __syncthreads();

        // ------------------------------- projection / back-projection matrices
        const int P16 = 16 * d.T;
        for (int e = t; e < P16 * 16; e += NTH) {
            const int i = e >> 4, g = e & 15;
            const bool ok = i < p && g < r;
            const double v = ok ? s_z[g][i] : 0.0;
            const double s = i < p ? s_sig[i] : 1.0;
            d.P32[e] = (float)(v / s);
            d.Q32[(int64_t)g * P16 + i] = (float)(v * s);
            if (ok) {
                d.P64[(int64_t)i * r + g] = v / s;
                d.Q64[(int64_t)g * p + i] = v * s;
            }
        }
        if (d.eig_check) {
            // accuracy of the computed eigenpairs of C = D^-1 G D^-1 (G is intact):
            // ||C V - V Lambda||_F / ||C||_F and max |V^T V - I| over the kr used
            double rs = 0.0, cs = 0.0, os = 0.0;
            for (int e = t; e < p * kr; e += NTH) {
                const int g = e / p, i = e - g * p;
                const double* gi = d.G + (int64_t)i * p;
                const double si = s_sig[i];
                double acc = 0.0;
                for (int j = 0; j < p; ++j) acc = fma(gi[j] / (si * s_sig[j]), s_z[g][j], acc);
                const double res = fma(-s_ev[g], s_z[g][i], acc);
                rs = fma(res, res, rs);
            }
            for (int e = t; e < p * p; e += NTH) {
                const int i = e / p, j = e - i * p;
                const double c = d.G[e] / (s_sig[i] * s_sig[j]);
                cs = fma(c, c, cs);
            }
            for (int e = t; e < kr * kr; e += NTH) {
                const int g = e / kr, k = e - g * kr;
                double dot = 0.0;
                for (int i = 0; i < p; ++i) dot = fma(s_z[g][i], s_z[k][i], dot);
                os = fmax(os, fabs(dot - (g == k ? 1.0 : 0.0)));
            }
            rs = wave_sum(rs);
            cs = wave_sum(cs);
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) os = fmax(os, __shfl_xor(os, o, 64));
            if (lane == 0) {
                s_chk[0][wave] = rs;
                s_chk[1][wave] = cs;
                s_chk[2][wave] = os;
            }
            __syncthreads();
            if (t == 0) {
                double a = 0.0, b = 0.0, m = 0.0;
                for (int w = 0; w < NW; ++w) {
                    a += s_chk[0][w];
                    b += s_chk[1][w];
                    m = fmax(m, s_chk[2][w]);
                }
                d.eig_check[0] = b > 0.0 ? sqrt(a / b) : 0.0;
                d.eig_check[1] = m;
            }
        }
        if (t == 0) {
            double gp = __builtin_inf();
            if (kr < p) {
                gp = s_ev[kr - 1] / s_ev[kr];
                if (!(gp >= 1.0 + 1e-6)) flags |= HYRES_DEV_DEGENERATE;
            }
            d.gap[0] = gp;
            if (d.rank_out) *d.rank_out = kr;
        }
    }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();
    if (t == 0 && s_flags) set_status(d.status, s_flags);
    HYRES_STAMP(d, 7);
}

// Gauss-Jordan sweep of the symmetric positive definite p x p matrix M held
// in the register tile A (thread (tr, tc) of the ROWS x COLS grid holds the
// entries (tr + ROWS a, tc + COLS b); entries beyond p hold the identity).
// Afterwards A = -M^-1.  diag: the diagonal of M in LDS, for the pivot test (a
// pivot below 1e-12 of its diagonal entry is replaced by 1 and reported as
// HYRES_DEV_NOT_PD).  Every thread of the block takes part (barriers).
template <int BR, int BC, int ROWS, int COLS>
__device__ __forceinline__ int gj_sweep(double (&A)[BR][BC], int p, int tr, int tc, const double* diag,
                                        double (*s_col)[kSmallP], double (*s_col2)[kSmallP]) {
    constexpr int NTH = ROWS * COLS;
    int flags = 0;
    // pivots in pairs (k0, k1): one barrier per pair.  The column k1 after
    // the k0 step is formed from the two broadcast columns exactly as the
    // k0 step forms it in the registers of its owners, so the result is
    // that of sweeping the pivots one at a time.  Grids of more than 512
    // threads (a tighter register budget) sweep one pivot per barrier.
    constexpr bool kPairs = NTH <= 512;
#pragma unroll
    for (int bb = 0; bb < BC; ++bb) {
        for (int kk = 0; kk < COLS; kk += kPairs ? 2 : 1) {
            const int k0 = COLS * bb + kk, k1 = k0 + 1;
            if (k0 >= p) break;
            const bool two = kPairs && k1 < p;
            const int buf = (kPairs ? k0 >> 1 : k0) & 1;
            if (tc == kk) {
#pragma unroll
                for (int a = 0; a < BR; ++a) s_col[buf][tr + ROWS * a] = A[a][bb];
            }
            if (two && tc == kk + 1) {
#pragma unroll
                for (int a = 0; a < BR; ++a) s_col2[buf][tr + ROWS * a] = A[a][bb];
            }
            __syncthreads();
            // the pivot is the regression residual of band k on the bands swept so far
            double d0 = s_col[buf][k0];
            if (!(d0 > 1e-12 * diag[k0])) {
                flags |= HYRES_DEV_NOT_PD;
                d0 = 1.0;
            }
            const double inv0 = 1.0 / d0;
            double cj[BC];
#pragma unroll
            for (int b = 0; b < BC; ++b) cj[b] = s_col[buf][tc + COLS * b];
#pragma unroll
            for (int a = 0; a < BR; ++a) {
                const int i = tr + ROWS * a;
                const double ci = s_col[buf][i] * inv0;
                if (i == k0) {
#pragma unroll
                    for (int b = 0; b < BC; ++b) A[a][b] = cj[b] * inv0;
                    if (tc == kk) A[a][bb] = -inv0;
                } else {
#pragma unroll
                    for (int b = 0; b < BC; ++b) A[a][b] = fma(-ci, cj[b], A[a][b]);
                    if (tc == kk) A[a][bb] = ci;
                }
            }
            if (two) {
                const double ck1 = s_col[buf][k1];
                // column k1 after the k0 step
                auto ep = [&](int i) {
                    return i == k0 ? ck1 * inv0 : fma(-(s_col[buf][i] * inv0), ck1, s_col2[buf][i]);
                };
                double d1 = ep(k1);
                if (!(d1 > 1e-12 * diag[k1])) {
                    flags |= HYRES_DEV_NOT_PD;
                    d1 = 1.0;
                }
                const double inv1 = 1.0 / d1;
#pragma unroll
                for (int b = 0; b < BC; ++b) cj[b] = ep(tc + COLS * b);
#pragma unroll
                for (int a = 0; a < BR; ++a) {
                    const int i = tr + ROWS * a;
                    const double ci = ep(i) * inv1;
                    if (i == k1) {
#pragma unroll
                        for (int b = 0; b < BC; ++b) A[a][b] = cj[b] * inv1;
                        if (tc == kk + 1) A[a][bb] = -inv1;
                    } else {
#pragma unroll
                        for (int b = 0; b < BC; ++b) A[a][b] = fma(-ci, cj[b], A[a][b]);
                        if (tc == kk + 1) A[a][bb] = ci;
                    }
                }
            }
        }
    }
    return flags;
}

// Eigen-adjoint systems (block k < r) and the inverse Gram (block r), one
// workgroup each, by the register sweep above.  For component k the system is
// (lambda_k I - C_perp) y = (I - U U^T) dV_k, C_perp = C - U Lambda U^T with the
// top r eigenpairs (U, Lambda) of C removed: it is symmetric positive
// definite (eigenvalue lambda_k on the top-r directions, lambda_k - lambda_i > 0
// on the others), so the sweep needs no pivoting.  y is the part of the
// eigenvector derivative outside the top-r subspace; inside it the derivative
// is explicit:  w_k = y + sum_{i<r, i!=k} u_i (u_i^T dV_k) / (lambda_k - lambda_i),
// the same w_k as the solution of (lambda_k I - C + lambda_k u_k u_k^T) w =
// (I - u_k u_k^T) dV_k.  dV_k = D^-1 dP_k + D dQ_k.
template <int BR, int BC, int ROWS, int COLS>
__global__ __launch_bounds__(ROWS * COLS) void k_adj_sweep(AdjDesc a) {
    constexpr int NTH = ROWS * COLS;
    constexpr int NW = NTH / 64;
    __shared__ double s_col[2][kSmallP];
    __shared__ double s_col2[2][kSmallP];
    __shared__ double s_diag[kSmallP], s_sig[kSmallP], s_rhs[kSmallP];
    __shared__ double s_u[kMaxRank][kSmallP];
    __shared__ double s_ev[kMaxRank], s_dot[kMaxRank];
    __shared__ double s_part[kSmallP][COLS];          // row partial sums of M^-1 rhs
    const int p = a.p, r = a.r, k = blockIdx.x;
    const int t = threadIdx.x, tc = t % COLS, tr = t / COLS, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    for (int i = t; i < p; i += NTH) s_sig[i] = a.sigma[i];
    for (int e = t; e < r * p; e += NTH) s_u[e / p][e % p] = a.V[e];
    if (t < r) s_ev[t] = a.evals[t];
    __syncthreads();
    const bool eig = k < r;
    const double lk = eig ? s_ev[k] : 0.0;
    if (eig) {
        for (int i = t; i < p; i += NTH) s_rhs[i] = a.dPt[(int64_t)k * p + i] / s_sig[i] + s_sig[i] * a.dQ[(int64_t)k * p + i];
        __syncthreads();
        for (int m = wave; m < r; m += NW) {
            double d = 0.0;
            for (int i = lane; i < p; i += 64) d = fma(s_u[m][i], s_rhs[i], d);
            d = wave_sum(d);
            if (lane == 0) s_dot[m] = d;
        }
        __syncthreads();
        for (int i = t; i < p; i += NTH) {
            double v = s_rhs[i];
            for (int m = 0; m < r; ++m) v = fma(-s_u[m][i], s_dot[m], v);
            s_rhs[i] = v;
            double dg = lk - a.G[(int64_t)i * p + i] / (s_sig[i] * s_sig[i]);
            for (int m = 0; m < r; ++m) dg = fma(s_ev[m] * s_u[m][i], s_u[m][i], dg);
            s_diag[i] = dg;
        }
    } else {
        for (int i = t; i < p; i += NTH) s_diag[i] = a.G[(int64_t)i * p + i];
    }
    double A[BR][BC];
#pragma unroll
    for (int aa = 0; aa < BR; ++aa)
#pragma unroll
        for (int b = 0; b < BC; ++b) {
            const int i = tr + ROWS * aa, j = tc + COLS * b;
            double v = i == j ? 1.0 : 0.0;
            if (i < p && j < p) {
                const double g = a.G[(int64_t)i * p + j];
                if (eig) {
                    v = (i == j ? lk : 0.0) - g / (s_sig[i] * s_sig[j]);
                    for (int m = 0; m < r; ++m) v = fma(s_ev[m] * s_u[m][i], s_u[m][j], v);
                } else {
                    v = g;
                }
            }
            A[aa][b] = v;
        }
    __syncthreads();
    const int flags = gj_sweep<BR, BC, ROWS, COLS>(A, p, tr, tc, s_diag, s_col, s_col2);
    if (flags && t == 0) set_status(a.status, flags);
    if (eig) {
        // y = M^-1 rhs = -A rhs: partial sums over this thread's columns, then rows in column order
#pragma unroll
        for (int aa = 0; aa < BR; ++aa) {
            double part = 0.0;
#pragma unroll
            for (int b = 0; b < BC; ++b) {
                const int j = tc + COLS * b;
                part = fma(A[aa][b], j < p ? s_rhs[j] : 0.0, part);
            }
            s_part[tr + ROWS * aa][tc] = part;
        }
        __syncthreads();
        for (int i = t; i < p; i += NTH) {
            double y = 0.0;
            for (int c = 0; c < COLS; ++c) y -= s_part[i][c];
            for (int m = 0; m < r; ++m)
                if (m != k) y = fma(s_u[m][i], s_dot[m] / (lk - s_ev[m]), y);
            a.Wsol[(int64_t)k * p + i] = y;
        }
    } else {
#pragma unroll
        for (int aa = 0; aa < BR; ++aa)
#pragma unroll
            for (int b = 0; b < BC; ++b) {
                const int i = tr + ROWS * aa, j = tc + COLS * b;
                if (i < p && j < p) a.Ginv[(int64_t)i * p + j] = -A[aa][b];
            }
    }
}

hipError_t launch_adj_sweep(const AdjDesc& a, hipStream_t s) {
    const int p = a.p;
    const dim3 grid(a.r + 1);
#define HYRES_A(BR, BC, RW, CL) hipLaunchKernelGGL((k_adj_sweep<BR, BC, RW, CL>), grid, dim3(RW * CL), 0, s, a)
    if (p <= 32) HYRES_A(2, 2, 16, 16);
    else if (p <= 64) HYRES_A(4, 4, 16, 16);
    else if (p <= 96) HYRES_A(6, 6, 16, 16);
    else if (p <= 128) HYRES_A(8, 8, 16, 16);
    else if (p <= 144) HYRES_A(5, 9, 32, 16);
    else if (p <= 160) HYRES_A(5, 10, 32, 16);
    else if (p <= 176) HYRES_A(11, 6, 16, 32);
    else if (p <= 192) HYRES_A(8, 6, 24, 32);
    else if (p <= 224) HYRES_A(7, 7, 32, 32);
    else return hipErrorInvalidValue;
#undef HYRES_A
    return hipGetLastError();
}

// Kernel variant of the class of up to p bands: T = p / 16 column tiles.
hipError_t launch_small(int p, const CubeDesc* descs, const int* cubes, int ncls, hipStream_t s) {
    switch ((p + 15) / 16) {
#define HYRES_S(T) \
    case T: hipLaunchKernelGGL(k_small<T>, dim3(ncls), dim3(64 * Cols<T>::NW), 0, s, descs, cubes, ncls); break;
        HYRES_S(1) HYRES_S(2) HYRES_S(4) HYRES_S(6) HYRES_S(8) HYRES_S(9) HYRES_S(10) HYRES_S(11) HYRES_S(12)
        HYRES_S(14)
#undef HYRES_S
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace hyres
