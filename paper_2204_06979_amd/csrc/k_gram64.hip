// Band Gram of FP64 cubes.
#include <algorithm>

#include "hyres_internal.hpp"

namespace hyres {

// FP64 Gram on the FP64 matrix cores.  A unit is a 32 x 32 block of G on or
// above the diagonal (2 x 2 tiles of 16 bands); a wave owns one unit of one slot
// (a run of pixels): element (pixel k, band m) of a 16-band fragment is the lane
// layout of both MFMA operands, so four loads of four pixels feed four products
// (two loads and three products on the diagonal), read eight steps ahead.  The
// four waves of a block are the quadrants of a 64 x 64 block of G, so that they
// share cache lines.
// The floor is the FP64 matrix rate (n p (p + 1) flops at 74 TFLOP/s); what
// bounds it is the cube coming in once per 64 x 64 block (256 x 256 x 128: 49 us,
// 5.5 TB/s of such reads; more or fewer waves, and a slot's blocks on one XCD,
// measured 49-67 us).  Before, one thread per entry of G walked the pixels of its
// slot: 552 us (64 x 64 x 32, now 6.5) and 1198 us (256 x 256 x 128).
// A band slot beyond p reads band p - 1: an entry of G depends on its own two
// bands only, and those beyond p are never written.
constexpr int kGram64Steps = 8;

// LINEAR: the pixels of the cube are a single run (row_pitch = W pitch), so whole
// groups of steps are read at a scalar base plus a constant lane offset; the
// per-lane walk over image rows costs more issue slots than the products.
template <bool DIAG, bool LINEAR>
__device__ __forceinline__ void gram_f64_unit(const CubeDesc& d, int I, int J, int64_t q0, int64_t q1, double* out) {
    const int lane = threadIdx.x & 63, col = lane & 15, kg = lane >> 4;
    const int pm = d.p - 1;
    constexpr int NF = DIAG ? 2 : 4, ST = kGram64Steps;
    const int band[4] = {min(32 * I + col, pm), min(32 * I + 16 + col, pm), min(32 * J + col, pm),
                         min(32 * J + 16 + col, pm)};
    int bad = 0;
    v4d acc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = (v4d){0.0, 0.0, 0.0, 0.0};
    auto step = [&](const double (&f)[NF]) {
        acc[0] = mfma4d(f[0], f[NF - 2], acc[0]);
        acc[1] = mfma4d(f[0], f[NF - 1], acc[1]);
        if constexpr (DIAG) bad |= !__builtin_isfinite(f[0]) || !__builtin_isfinite(f[1]);
        else acc[2] = mfma4d(f[1], f[2], acc[2]);
        acc[3] = mfma4d(f[1], f[NF - 1], acc[3]);
    };
    auto steps = [&](const double (&f)[ST][NF]) {
#pragma unroll
        for (int s = 0; s < ST; ++s) step(f[s]);
    };
    double cur[ST][NF], nxt[ST][NF];
    int64_t b = q0;
    if constexpr (LINEAR) {
        uint32_t off[NF];
#pragma unroll
        for (int k = 0; k < NF; ++k) off[k] = (uint32_t)(kg * d.pitch + band[k]);
        auto fetch = [&](double (&f)[ST][NF], int64_t q) {
            const HYRES_GLOBAL double* y = gmem(static_cast<const double*>(d.Y)) + q * d.pitch;
#pragma unroll
            for (int s = 0; s < ST; ++s)
#pragma unroll
                for (int k = 0; k < NF; ++k) f[s][k] = (y + 4 * s * d.pitch)[off[k]];
        };
        if (b + 4 * ST <= q1) fetch(cur, b);
        while (b + 4 * ST <= q1) {
            if (b + 8 * ST <= q1) fetch(nxt, b + 4 * ST);
            steps(cur);
            b += 4 * ST;
            if (b + 4 * ST > q1) break;
            if (b + 8 * ST <= q1) fetch(cur, b + 4 * ST);
            steps(nxt);
            b += 4 * ST;
        }
    }
    // groups of steps with a pointer per lane, pixels beyond the slot as zeros
    for (; b < q1; b += 4 * ST) {
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            const int64_t q = min(b + 4 * s + kg, q1 - 1);
            const HYRES_GLOBAL double* y = gmem(pixel_ptr<double>(d, q));
#pragma unroll
            for (int k = 0; k < NF; ++k) cur[s][k] = y[band[k]];
        }
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            double f[NF];
#pragma unroll
            for (int k = 0; k < NF; ++k) f[k] = b + 4 * s + kg < q1 ? cur[s][k] : 0.0;
            step(f);
        }
    }
    if (bad) set_status(d.status, HYRES_DEV_NONFINITE);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int v = 0; v < 4; ++v) gmem(out)[k * 256 + v * 64 + lane] = acc[k][v];
}

// Units and 64 x 64 blocks of G on or above the diagonal.
__host__ __device__ inline int gram_f64_units(int T) {
    const int T2 = (T + 1) / 2;
    return T2 * (T2 + 1) / 2;
}
__host__ __device__ inline int gram_f64_blocks(int T) {
    const int T4 = (T + 3) / 4;
    return T4 * (T4 + 1) / 2;
}

__global__ __launch_bounds__(256) void k_gram_f64(const CubeDesc* __restrict__ descs, int cube) {
    const CubeDesc& d = descs[cube];
    const int T2 = (d.T + 1) / 2, units = gram_f64_units(d.T);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int64_t per = (d.n + d.gslots - 1) / d.gslots;
    per = (per + 4 * kGram64Steps - 1) / (4 * kGram64Steps) * (4 * kGram64Steps);
    int slot, I = 0, J = 0;
    if (T2 == 1) {                            // one unit: the waves take slots of their own
        slot = blockIdx.x * 4 + wave;
    } else {
        const int blocks = gram_f64_blocks(d.T), T4 = (d.T + 3) / 4;
        slot = blockIdx.x / blocks;
        int I4 = 0, rem = blockIdx.x - slot * blocks;
        while (rem >= T4 - I4) { rem -= T4 - I4; ++I4; }
        I = 2 * I4 + (wave >> 1);
        J = 2 * (I4 + rem) + (wave & 1);
    }
    if (slot >= d.gslots || I > J || J >= T2) return;
    const int64_t q0 = min((int64_t)slot * per, d.n), q1 = min(q0 + per, d.n);
    const int u = I * T2 - I * (I - 1) / 2 + (J - I);
    double* out = static_cast<double*>(d.gpart) + ((int64_t)slot * units + u) * 1024;
    if (d.row_pitch == d.W * d.pitch) {
        if (I == J) gram_f64_unit<true, true>(d, I, J, q0, q1, out);
        else gram_f64_unit<false, true>(d, I, J, q0, q1, out);
    } else {
        if (I == J) gram_f64_unit<true, false>(d, I, J, q0, q1, out);
        else gram_f64_unit<false, false>(d, I, J, q0, q1, out);
    }
}

// Sums the slots' partials of 16 entries of one tile: 16 threads per entry take
// every 16th slot, then the 16 sums are added in order.
__global__ __launch_bounds__(256) void k_gram_reduce_f64(const CubeDesc* __restrict__ descs, int cube) {
    __shared__ double s_sum[16][17];
    const CubeDesc& d = descs[cube];
    const int T2 = (d.T + 1) / 2, units = gram_f64_units(d.T);
    const int tile = blockIdx.x >> 4, u = tile >> 2, tt = tile & 3;
    int I = 0, rem = u;
    while (rem >= T2 - I) { rem -= T2 - I; ++I; }
    const int bi = 2 * I + (tt >> 1), bj = 2 * (I + rem) + (tt & 1);
    if (bi > bj || bj >= d.T) return;
    const int es = threadIdx.x & 15, sl = threadIdx.x >> 4;
    const int e = (blockIdx.x & 15) * 16 + es;
    const HYRES_GLOBAL double* part = gmem(static_cast<const double*>(d.gpart)) + (int64_t)u * 1024 + tt * 256 + e;
    double s = 0.0;
#pragma unroll 8
    for (int k = sl; k < d.gslots; k += 16) s += part[(int64_t)k * units * 1024];
    s_sum[sl][es] = s;
    __syncthreads();
    if (sl) return;
    s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) s += s_sum[k][es];
    const int lane = e & 63, v = e >> 6;
    const int a = 16 * bi + (lane >> 4) + 4 * v, b = 16 * bj + (lane & 15);
    if (a < d.p && b < d.p && a <= b) {
        d.G[(int64_t)a * d.p + b] = s;
        d.G[(int64_t)b * d.p + a] = s;
    }
}

// Slots of an FP64 Gram: about two waves per SIMD of a full chip (512 blocks), at
// least 64 pixels each, and no more slots than the reduce adds in a few
// microseconds (512).
int gram_f64_slots(int T, int64_t n) {
    const int b = gram_f64_blocks(T);
    int64_t slots = std::min<int64_t>(512, (512 + b - 1) / b);
    slots = std::min<int64_t>(slots, (n + 63) / 64);
    return (int)std::max<int64_t>(1, slots);
}
size_t gram_f64_bytes(int T, int slots) { return (size_t)slots * gram_f64_units(T) * 1024 * sizeof(double); }

hipError_t launch_gram_f64(const CubeDesc* descs, int cube, int p, int gslots, hipStream_t s) {
    const int T = (p + 15) / 16;
    const int grid = T <= 2 ? (gslots + 3) / 4 : gram_f64_blocks(T) * gslots;
    hipLaunchKernelGGL(k_gram_f64, dim3(grid), dim3(256), 0, s, descs, cube);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_reduce_f64, dim3(gram_f64_units(T) * 64), dim3(256), 0, s, descs, cube);
    return hipGetLastError();
}

}  // namespace hyres
