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
// The p x p matrix lives in registers by columns (T = ceil(p / 16) column
// tiles): lane (g, c) = (lane / 16, lane mod 16) of the wave that owns column
// tile w holds, of column 16 w + c, the rows 4 e + g, e < 4 T.  A vector that
// multiplies the rows is read from LDS as T / 4 registers, lane (g, c) holding its
// entries of rows 4 (16 m + c) + g, and a product with row 4 (16 m + c') + g takes
// the entry of lane c' of the same 16 lanes as its operand (row_newbcast of
// v_fmac_f64): one instruction per entry and no LDS traffic or register for the
// row operand.  Column sums stay in the lane but for two swaps over g, and a
// matrix row, which by symmetry is the next column, leaves the registers with
// one LDS write per wave.  From T = 5 on a wave owns the tiles w and w + W
// (W = ceil(T / 2)): the work of a step beside the products (norm, square root,
// quotient, reductions) is issued once for both, and no SIMD has more than two
// waves.  Both eliminations are bound by instruction issue, the late steps of the
// tridiagonalisation by the latency of its two barriers and its square root.
// The previous layout (a thread grid with 5 x 9 entries per thread at p = 144,
// row sums over 16 lanes by DPP, the operands of both sides from LDS) issued
// about 480 vector instructions per Householder step and wave.
#include "hyres_internal.hpp"

namespace hyres {

constexpr int kSmallP = 256;   // LDS vector length (p <= 224)

// Sturm count: number of eigenvalues of the symmetric tridiagonal matrix
// smaller than x, from the sign changes of the leading principal minors
// p_i(x) = (d_i - x) p_{i-1}(x) - e_{i-1}^2 p_{i-2}(x) (a minor that is
// exactly zero counts as positive); both minors are rescaled by a power of two
// every 8 steps so the recursion stays in range.  de[i] = (d_i, e_{i-1}^2), a
// step is three FP64 instructions and one that shifts the sign into a word; the
// next 8 entries are read while these run.
__device__ __forceinline__ int sgnbit(double v) { return (int)((unsigned)__double2hiint(v) >> 31); }

__device__ __forceinline__ int sturm_count(const double2* __restrict__ de, int p, double x) {
    double pm2 = 1.0, pm1 = de[0].x - x;
    uint32_t bits = (uint32_t)sgnbit(pm1);     // signs of the minors, the latest lowest
    int cnt = (int)bits, i = 1;
    double2 cur[8];
    if (i + 8 <= p) {
#pragma unroll
        for (int u = 0; u < 8; ++u) cur[u] = de[i + u];
    }
    for (; i + 8 <= p; i += 8) {
        double2 nxt[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) nxt[u] = de[i + 8 + u];      // past p: padding, not used
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double pi = fma(cur[u].x - x, pm1, -cur[u].y * pm2);
            bits = __builtin_amdgcn_alignbit(bits, (uint32_t)__double2hiint(pi), 31);
            pm2 = pm1;
            pm1 = pi;
        }
        cnt += __builtin_popcount((bits ^ (bits >> 1)) & 0xffu);
        const int e1 = __builtin_amdgcn_frexp_exp(pm1), e2 = __builtin_amdgcn_frexp_exp(pm2);
        const int e = e1 > e2 ? e1 : e2;
        pm1 = ldexp(pm1, -e);
        pm2 = ldexp(pm2, -e);
#pragma unroll
        for (int u = 0; u < 8; ++u) cur[u] = nxt[u];
    }
    for (int u = 0; i < p; ++i, ++u) {
        const double2 v = de[i];
        const double pi = fma(v.x - x, pm1, -v.y * pm2);
        bits = __builtin_amdgcn_alignbit(bits, (uint32_t)__double2hiint(pi), 31);
        cnt += (int)((bits ^ (bits >> 1)) & 1u);
        pm2 = pm1;
        pm1 = pi;
    }
    return cnt;
}

// In place: lo = max and hi = min over each aligned group of M lanes (M = 4, 16, 32 or 64).
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
    if (M == 32) {
        const bool upper = (threadIdx.x & 32) != 0;
        lo = upper ? lb : la;
        hi = upper ? hb : ha;
        return;
    }
    lo = la > lb ? la : lb;
    hi = ha < hb ? ha : hb;
}

// ---- products of register rows with a vector held in lanes (see the top) ----
// a[k] += x[lane C0 + k of this row of 16] * z, k < N.  The wait states at the
// start cover a write of x right before (a DPP operand needs two).
#define HYRES_BC(A, X, Z, C) "v_fmac_f64_dpp " A ", " X ", " Z " row_newbcast:" C " row_mask:0xf bank_mask:0xf\n"
template <int E0, int N, int E>
__device__ __forceinline__ void axpy_block(double (&a)[E], double x, double z) {
    constexpr int C0 = E0 & 15;
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
template <int E0, int N, int E>
__device__ __forceinline__ void dot_block(const double (&a)[E], double x, double (&y)[4]) {
    constexpr int C0 = E0 & 15;
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
// All rows from element E0 on.
template <int E0, int E, int M>
__device__ __forceinline__ void axpy_rows(double (&a)[E], const double (&x)[M], double z) {
    if constexpr (E0 < E) {
        constexpr int room = 16 - (E0 & 15), len = room < E - E0 ? room : E - E0;
        constexpr int N = len >= 16 ? 16 : len >= 8 ? 8 : 4;
        axpy_block<E0, N>(a, x[E0 >> 4], z);
        axpy_rows<E0 + N, E, M>(a, x, z);
    }
}
template <int E0, int E, int M>
__device__ __forceinline__ void dot_rows(const double (&a)[E], const double (&x)[M], double (&y)[4]) {
    if constexpr (E0 < E) {
        constexpr int room = 16 - (E0 & 15), len = room < E - E0 ? room : E - E0;
        constexpr int N = len >= 8 ? 8 : 4;
        dot_block<E0, N>(a, x[E0 >> 4], y);
        dot_rows<E0 + N, E, M>(a, x, y);
    }
}

// Sum over the four rows of 16 lanes, to every lane.
__device__ __forceinline__ double rows_sum(double v) {
    {
        const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
    }
    const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}

// a[E0 + q] for the wave-uniform q < N (every index a constant: the array stays in
// registers).
template <int E0, int N, int E>
__device__ __forceinline__ double pick(const double (&a)[E], int q) {
    if constexpr (N > 1 && E0 + N > E) {
        return pick<E0, N - 1, E>(a, q);
    } else if constexpr (N == 1) {
        return a[E0];
    } else {
        const double v = pick<E0, N - 1, E>(a, q);
        return q == N - 1 ? a[E0 + N - 1] : v;
    }
}

// Shape of the column layout of T tiles.
template <int T>
struct Cols {
    static constexpr int NC = T >= 5 ? 2 : 1;            // column tiles per wave
    static constexpr int W = (T + NC - 1) / NC;          // waves that own columns
    static constexpr int NW = T >= 5 ? 8 : 4;            // waves of the block
    static constexpr int E = 4 * T;                      // rows per lane
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
    constexpr int NW = CL::NW, NTH = 64 * NW, NC = CL::NC, W = CL::W, E = CL::E, M = CL::M, SP = CL::SP;
    constexpr int Q = CL::Q, PL = CL::PL;
    constexpr int VPW = (kMaxRank + NW - 1) / NW;   // eigenvectors per wave
    if ((int)blockIdx.x >= ncls) return;
    const CubeDesc& d = descs[cubes[blockIdx.x]];
    const int p = d.p, r = d.r;
    const double nn = (double)d.n;
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    __shared__ double s_row[2][2][4 * SP];           // matrix rows on their way (noise: pairs)
    __shared__ double s_u[4 * SP];
    __shared__ double s_col[2][PL];
    __shared__ double s_sig[PL];
    __shared__ double s_dd[PL], s_ee[PL], s_hb[PL], s_ev[PL];
    __shared__ double2 s_de[PL + 16];                // scaled (d_i, e_{i-1}^2)
    __shared__ double s_zL[PL * kMaxRank];           // multipliers of the top-down factorisation [i][g]
    __shared__ double s_zU[PL * kMaxRank];           // multipliers of the bottom-up one         [i][g]
    __shared__ double s_z[kMaxRank][PL];             // eigenvectors of the tridiagonal / of C
    __shared__ double s_red[4];
    __shared__ double s_vav[NW];                     // per-wave shares of v^T A v
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
    double A[NC][E];
    // column and slot of this lane per column tile (tiles beyond T: column -1)
    int col[NC], own[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
        const int tile = wave + W * j;
        col[j] = wave < W && tile < T ? 16 * tile + c : -1;
        own[j] = col[j] >= 0 ? slot_of<T>(col[j]) : 0;
    }
    const HYRES_GLOBAL double* G = gmem(static_cast<const double*>(d.G));
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
            static_for<NC * E>([&](auto x) {
                constexpr int j = decltype(x)::value / E, e = decltype(x)::value % E;
                const int i = 4 * e + g, n = col[j];
                A[j][e] = i < p && n >= 0 && n < p ? G[(int64_t)i * p + n] : (i == n ? 1.0 : 0.0);
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
            for (int kk = 0; kk < 16; kk += 2) {
                const int k0 = 16 * t0 + kk, k1 = k0 + 1;
                if (k0 >= p) break;
                double (*row)[4 * SP] = s_row[(kk >> 1) & 1];
                const int gr = g - (kk & 3);             // 0: holds row k0, 1: row k1
                if (wave < W) {
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const double v = pick<4 * t0, 4>(A[j], kk >> 2);
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
                const double inv0 = 1.0 / d0, m01 = r01 * inv0;
                double d1 = fma(-r01, m01, r11);
                if (!(d1 > 1e-12 * s_ev[k1])) {
                    flags |= HYRES_DEV_NOT_PD;
                    d1 = 1.0;
                }
                const double inv1 = 1.0 / d1;
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
                        axpy_rows<4 * t0, E, M>(A[j], x0, -c0);
                        axpy_rows<4 * t0, E, M>(A[j], x1, -c1);
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
            static_for<NC * E>([&](auto x) {
                constexpr int j = decltype(x)::value / E, e = decltype(x)::value % E;
                const int i = 4 * e + g, n = col[j];
                A[j][e] = i < p && n >= 0 && n < p ? G[(int64_t)i * p + n] / (s_sig[i] * s_sig[n]) : 0.0;
            });
        }
        for (int i = t; i < 4 * SP; i += NTH) s_row[0][0][i] = s_row[1][0][i] = 0.0;
        __syncthreads();

        // ------------------------------------------------ tridiagonalisation
        // Step k, x the entries of row k beyond the diagonal: v = x - alpha e_{k+1},
        // u = beta A v, A <- A - v w^T - w v^T with w = u - K v, K = (beta / 2) u^T v, that
        // is A_in -= v_i (u_n - 2 K v_n) + u_i v_n.  A v = A x - alpha A e_{k+1}: the
        // products with x do not wait for the norm that gives alpha.
        static_for<T>([&](auto tc) {
            constexpr int t0 = decltype(tc)::value, m0 = t0 / 4;
            for (int kk = 0; kk < 16; ++kk) {
                const int k = 16 * t0 + kk;
                if (k >= p - 2) break;
                double* xs = s_row[k & 1][0];
                bool act[NC], any = false;
                static_for<NC>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    const int tile = wave + W * j;
                    const bool has = wave < W && tile < T;
                    act[j] = has && tile >= t0;
                    any |= act[j];
                    // row k; zeros up to the diagonal (the tile before t0 clears its last entry)
                    if (has && tile >= t0 - 1) {
                        const double v = pick<4 * t0, 4>(A[j], kk >> 2);
                        if (g == (kk & 3)) {
                            xs[own[j]] = col[j] > k ? v : 0.0;
                            if (col[j] == k) s_dd[k] = v;
                        }
                    }
                });
                __syncthreads();
                double xr[M], u[NC], v[NC], alpha = 0.0, beta = 0.0;
                if (any) {
                    double ss = 0.0;
#pragma unroll
                    for (int m = m0; m < M; ++m) {
                        xr[m] = xs[g * SP + 16 * m + c];
                        ss = fma(xr[m], xr[m], ss);
                    }
                    const double x1 = xs[slot_of<T>(k + 1)];
                    double y[NC];
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        y[j] = 0.0;
                        if (act[j]) {
                            double q[4] = {0.0, 0.0, 0.0, 0.0};
                            dot_rows<4 * t0, E, M>(A[j], xr, q);
                            y[j] = (q[0] + q[1]) + (q[2] + q[3]);
                        }
                    });
                    ss = rows_sum(row16_sum(ss));
                    const double nrm = sqrt(ss);
                    alpha = x1 >= 0.0 ? -nrm : nrm;
                    const double vtv = 2.0 * alpha * (alpha - x1);
                    beta = vtv > 0.0 ? 2.0 / vtv : 0.0;
                    const double v1 = x1 - alpha;
                    // v in place of x: the lane that holds entry k + 1
                    {
                        const bool mine = lane == ((k + 1) & 3) * 16 + (((k + 1) >> 2) & 15);
                        if ((t0 & 3) == 3 && t0 + 1 < T && kk == 15) {
                            constexpr int m1 = m0 + 1 < M ? m0 + 1 : m0;
                            xr[m1] = mine ? v1 : xr[m1];
                        } else {
                            xr[m0] = mine ? v1 : xr[m0];
                        }
                    }
                    const bool row1 = g == ((kk + 1) & 3);
                    double q = 0.0;
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        u[j] = v[j] = 0.0;
                        if (act[j]) {
                            const double a1 = pick<4 * t0, 5>(A[j], (kk + 1) >> 2);
                            y[j] = rows_sum(row1 ? fma(-alpha, a1, y[j]) : y[j]);
                            v[j] = col[j] == k + 1 ? v1 : xs[own[j]];
                            q = fma(v[j], y[j], q);
                            u[j] = beta * y[j];
                            if (g == 0) s_u[own[j]] = u[j];
                            if (g == 1 && col[j] > k && col[j] < p) d.hv[(int64_t)k * p + col[j]] = v[j];
                        }
                    });
                    q = row16_sum(q);
                    if (lane == 0) s_vav[wave] = q;
                    if (col[0] == 16 * t0 + c || (NC == 2 && col[NC - 1] == 16 * t0 + c)) {   // the wave of tile t0
                        if (lane == 0) {
                            s_ee[k] = alpha;
                            s_hb[k] = beta;
                        }
                    }
                }
                __syncthreads();
                if (any) {
                    double vav = 0.0;
#pragma unroll
                    for (int w = 0; w < W; ++w)
                        if (w >= t0 || (NC == 2 && w + W < T && w + W >= t0)) vav += s_vav[w];
                    const double K2 = beta * (beta * vav);
                    double ur[M];
#pragma unroll
                    for (int m = m0; m < M; ++m) ur[m] = s_u[g * SP + 16 * m + c];
                    static_for<NC>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        if (act[j]) {
                            axpy_rows<4 * t0, E, M>(A[j], xr, fma(K2, v[j], -u[j]));
                            axpy_rows<4 * t0, E, M>(A[j], ur, -v[j]);
                        }
                    });
                }
            }
        });
        __syncthreads();
        constexpr int EL = E > 8 ? 8 : E;                // rows of the last two tiles
        static_for<NC * EL>([&](auto x) {
            constexpr int j = decltype(x)::value / EL, e = E - EL + decltype(x)::value % EL;
            const int i = 4 * e + g, n = col[j];
            if (i == n && i >= p - 2 && i < p) s_dd[i] = A[j][e];
            if (i == p - 1 && n == p - 2) s_ee[p - 2] = A[j][e];
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
        for (int i = t; i < PL + 16; i += NTH) {
            const double es = i > 0 && i < p ? s_ee[i - 1] * sc : 0.0;
            s_de[i] = make_double2(i < p ? s_dd[i] * sc : 0.0, es * es);
        }
        __syncthreads();
        // Multisection: M lanes per eigenvalue evaluate the Sturm count at M
        // interior points, shrinking the bracket M+1 times per iteration.
        // Only the top r+1 eigenvalues are needed by the solve; all p are
        // computed when requested.
        {
            const int nev = (d.mode & 16) ? p : (r + 1 < p ? r + 1 : p);
            const int M = nev * 64 <= NTH ? 64 : (nev * 16 <= 2 * NTH ? 16 : 4);
            const int iters = M == 64 ? 9 : (M == 16 ? 14 : 24);
            const double inv_m1 = 1.0 / (double)(M + 1);
            const int m = t % M;
            const int nslot = NTH / M;
            for (int g0 = 0; g0 < nev; g0 += nslot) {
                const int g = g0 + t / M;
                if (g < nev) {
                    const int midx = p - 1 - g;        // ascending index of the g-th largest
                    double lo = -1.0 - 1e-12, hi = 1.0 + 1e-12;
                    for (int it = 0; it < iters; ++it) {
                        const double x = lo + (hi - lo) * ((double)(m + 1) * inv_m1);
                        const int cnt = sturm_count(s_de, p, x);
                        const bool below = cnt <= midx;   // x <= lambda
                        double lo_c = below ? x : lo;
                        double hi_c = below ? hi : x;
                        // largest lower and smallest upper end over the M lanes of
                        // the group: quads and rows by DPP, whole waves by readlane
                        group_maxmin(lo_c, hi_c, M);
                        lo = lo_c;
                        hi = hi_c;
                    }
                    if (m == 0) {
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
        // Reflectors are staged from global memory into LDS eight at a time by
        // the whole block (coalesced), then applied by the waves owning vectors.
        {
            constexpr int RB = 8;
            constexpr int SPT = (RB * PL + NTH - 1) / NTH;   // staged entries per thread
            double* stage = s_zL;                       // free now: RB x PL doubles
            // the next group's reflectors are read into registers while the
            // current group is applied
            double nxt[SPT];
            auto fetch = [&](int k1) {
                const int k0 = k1 - RB + 1 < 0 ? 0 : k1 - RB + 1;
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const int e = t + j * NTH;
                    const int kk = k1 - e / PL, i = e % PL;
                    nxt[j] = (e < RB * PL && kk >= k0 && i > kk && i < p) ? d.hv[(int64_t)kk * p + i] : 0.0;
                }
            };
            if (p - 3 >= 0) fetch(p - 3);
            for (int k1 = p - 3; k1 >= 0; k1 -= RB) {
                const int k0 = k1 - RB + 1 < 0 ? 0 : k1 - RB + 1;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < SPT; ++j) {
                    const int e = t + j * NTH;
                    if (e < RB * PL) stage[e] = nxt[j];
                }
                __syncthreads();
                if (k1 - RB >= 0) fetch(k1 - RB);
                if (wave < r) {
                    for (int k = k1; k >= k0; --k) {
                        const double* hk = stage + (k1 - k) * PL;
                        double h[Q];
#pragma unroll
                        for (int q = 0; q < Q; ++q) h[q] = hk[lane + 64 * q];
                        const double hb = s_hb[k];
#pragma unroll
                        for (int v = 0; v < VPW; ++v) {
                            if (wave + NW * v < r) {
                                double sdot = 0.0;
#pragma unroll
                                for (int q = 0; q < Q; ++q) sdot = fma(h[q], zr[v][q], sdot);
                                sdot = wave_sum(sdot) * hb;
#pragma unroll
                                for (int q = 0; q < Q; ++q) zr[v][q] = fma(-sdot, h[q], zr[v][q]);
                            }
                        }
                    }
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

// Kernel variant for p bands: T = ceil(p / 16) column tiles.
hipError_t launch_small(int p, const CubeDesc* descs, const int* cubes, int ncls, hipStream_t s) {
    switch ((p + 15) / 16) {
#define HYRES_S(T) \
    case T: hipLaunchKernelGGL(k_small<T>, dim3(ncls), dim3(64 * Cols<T>::NW), 0, s, descs, cubes, ncls); break;
        HYRES_S(1) HYRES_S(2) HYRES_S(3) HYRES_S(4) HYRES_S(5) HYRES_S(6) HYRES_S(7)
        HYRES_S(8) HYRES_S(9) HYRES_S(10) HYRES_S(11) HYRES_S(12) HYRES_S(13) HYRES_S(14)
#undef HYRES_S
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace hyres
