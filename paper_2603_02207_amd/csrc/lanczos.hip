// Lanczos recurrence of the spectral interval's upper end, two launches per
// step and no host round trip inside it.
//
// With u_j the unnormalised vector of step j and v_j = u_j / beta_{j-1}
// (beta_{-1} = 1), a step is
//     product:  w = A v_j,               partial sums of alpha_j = <v_j, w>
//     update:   u_{j+1} = w - alpha_j v_j - beta_{j-1} v_{j-1},
//               partial sums of beta_j^2 = <u_{j+1}, u_{j+1}>
// and each launch starts by adding up the partial sums of the one before it in
// every workgroup (at most kLanczosWgs doubles from L2, in a fixed order), so
// the scalars never leave the device while the recurrence runs.  All in FP64,
// an FP32 matrix's values widened as they are read.
//
// Bound by the latency of a row's reads (row pointer, column, gathered value)
// and the launches: 200000 rows of 15 entries, FP32, take 22 us per step; eight
// launches, two host round trips and one lane per row took 95 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.h"

namespace ld {

namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ void two_sum_into(double& s, double& c, double x) {
    const double t = s + x;
    c += fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s;
    s = t;
}

// Sum of p[0..count) in a fixed order (compensated), the same in every thread.
__device__ double sum_partials(const double* __restrict__ p, int count, double* sh) {
    double s = 0.0, c = 0.0;
    for (int i = threadIdx.x; i < count; i += kThreads) two_sum_into(s, c, p[i]);
    sh[threadIdx.x] = s;
    sh[kThreads + threadIdx.x] = c;
    __syncthreads();
    for (int h = kThreads / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            double a = sh[threadIdx.x], b = sh[kThreads + threadIdx.x] + sh[kThreads + threadIdx.x + h];
            two_sum_into(a, b, sh[threadIdx.x + h]);
            sh[threadIdx.x] = a;
            sh[kThreads + threadIdx.x] = b;
        }
        __syncthreads();
    }
    const double total = sh[0] + sh[kThreads];
    __syncthreads();
    return total;
}

__device__ double block_sum(double x, double* sh) {
    sh[threadIdx.x] = x;
    __syncthreads();
    for (int h = kThreads / 2; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    const double t = sh[0];
    __syncthreads();
    return t;
}

// u_0 = v_0: entries +-scale, the sign of SplitMix64 output row + 1 of the key
__global__ __launch_bounds__(kThreads) void lanczos_start_kernel(int n, uint64_t key, double scale,
                                                                 double* __restrict__ u) {
    for (int r = blockIdx.x * kThreads + threadIdx.x; r < n; r += gridDim.x * kThreads) {
        uint64_t z = key + ((uint64_t)r + 1ull) * 0x9E3779B97F4A7C15ull;
        z ^= z >> 30;
        z *= 0xBF58476D1CE4E5B9ull;
        z ^= z >> 27;
        z *= 0x94D049BB133111EBull;
        z ^= z >> 31;
        u[r] = (z >> 63) ? -scale : scale;
    }
}

// LPR lanes share a row's entries.
template <typename T, int LPR>
__global__ __launch_bounds__(kThreads) void lanczos_product_kernel(
    int n, const int* __restrict__ row_ptr, const int* __restrict__ col_idx, const T* __restrict__ val,
    const double* __restrict__ u, double* __restrict__ w, int j, const double* __restrict__ part_b, int parts,
    double* __restrict__ beta, double* __restrict__ part_a) {
    __shared__ double sh[2 * kThreads];
    double inv = 1.0;
    if (j > 0) {
        const double b = sqrt(fmax(sum_partials(part_b, parts, sh), 0.0));
        if (blockIdx.x == 0 && threadIdx.x == 0) beta[j - 1] = b;
        inv = 1.0 / b;
    }
    constexpr int kRows = kThreads / LPR;
    const int li = threadIdx.x % LPR, g = threadIdx.x / LPR;
    double dot = 0.0;
    for (int r0 = blockIdx.x * kRows; r0 < n; r0 += gridDim.x * kRows) {
        const int r = r0 + g;
        double s = 0.0;
        if (r < n) {
            const int end = row_ptr[r + 1];
#pragma unroll 4
            for (int k = row_ptr[r] + li; k < end; k += LPR) s = fma((double)val[k], u[col_idx[k]], s);
        }
#pragma unroll
        for (int h = LPR / 2; h >= 1; h >>= 1) s += __shfl_xor(s, h, 64);
        if (r < n && li == 0) {
            const double x = inv * s;
            w[r] = x;
            dot = fma(inv * u[r], x, dot);
        }
    }
    const double t = block_sum(dot, sh);
    if (threadIdx.x == 0) part_a[blockIdx.x] = t;
}

// w becomes u_{j+1}
__global__ __launch_bounds__(kThreads) void lanczos_update_kernel(int n, double* __restrict__ w,
                                                                  const double* __restrict__ u,
                                                                  const double* __restrict__ u_prev, int j,
                                                                  const double* __restrict__ beta,
                                                                  const double* __restrict__ part_a, int parts,
                                                                  double* __restrict__ alpha,
                                                                  double* __restrict__ part_b) {
    __shared__ double sh[2 * kThreads];
    const double a = sum_partials(part_a, parts, sh);
    if (blockIdx.x == 0 && threadIdx.x == 0) alpha[j] = a;
    const double b1 = j > 0 ? beta[j - 1] : 0.0;               // beta_{j-1}
    const double inv = j > 0 ? 1.0 / b1 : 1.0;                 // v_j = inv u_j
    const double inv_prev = j > 1 ? 1.0 / beta[j - 2] : 1.0;   // v_{j-1} = inv_prev u_{j-1}
    double sq = 0.0;
    for (int r = blockIdx.x * kThreads + threadIdx.x; r < n; r += gridDim.x * kThreads) {
        double x = fma(-a, inv * u[r], w[r]);
        if (j > 0) x = fma(-b1, inv_prev * u_prev[r], x);
        w[r] = x;
        sq = fma(x, x, sq);
    }
    const double t = block_sum(sq, sh);
    if (threadIdx.x == 0) part_b[blockIdx.x] = t;
}

__global__ __launch_bounds__(kThreads) void lanczos_beta_kernel(const double* __restrict__ part_b, int parts,
                                                                double* __restrict__ beta, int j) {
    __shared__ double sh[2 * kThreads];
    const double b = sqrt(fmax(sum_partials(part_b, parts, sh), 0.0));
    if (threadIdx.x == 0) beta[j] = b;
}

template <typename T>
void launch_product(const CsrDev& A, const LanczosDev& d, const double* u, double* w, int j, hipStream_t st) {
    // Lanes per row: 200000 rows of 15 entries took 1.62 ms for 64 steps with 4
    // lanes, 1.83 with 2, 1.76 with 8, 2.00 with 16 (fewer rows in flight); long
    // rows take 16.  (On average: a single long row is walked by its lanes alone.
    // 200000 rows, three of them with as many entries, take 360 ms for 64 steps, 1640
    // with one lane per row; a random graph of 2^20 rows and 17 entries 14.1, 48.8.)
    // Workgroups: 2048 against 1024 (1.94 ms at 8 lanes) and 3072
    // (2.27 ms at 4: more partial sums than the added rows in flight are worth).
    const long long avg = A.n > 0 ? (long long)A.nnz / A.n : 0;
#define LD_LZ(LPR_)                                                                                              \
    hipLaunchKernelGGL((lanczos_product_kernel<T, LPR_>), dim3(d.wgs), dim3(kThreads), 0, st, A.n, A.row_ptr,    \
                       A.col_idx, (const T*)A.val, u, w, j, d.part_b, d.wgs, d.beta, d.part_a)
    if (avg <= 24)
        LD_LZ(4);
    else
        LD_LZ(16);
#undef LD_LZ
}

}  // namespace

int lanczos_wgs(int n) { return std::max(1, std::min((n + 63) / 64, kLanczosWgs)); }

hipError_t launch_lanczos_start(int n, uint64_t key, double scale, double* u, hipStream_t st) {
    hipLaunchKernelGGL(lanczos_start_kernel, dim3(std::max(1, std::min((n + kThreads - 1) / kThreads, 2048))),
                       dim3(kThreads), 0, st, n, key, scale, u);
    return hipGetLastError();
}

hipError_t launch_lanczos_step(bool f64, const CsrDev& A, const LanczosDev& d, const double* u, const double* u_prev,
                               double* w, int j, hipStream_t st) {
    if (f64)
        launch_product<double>(A, d, u, w, j, st);
    else
        launch_product<float>(A, d, u, w, j, st);
    hipLaunchKernelGGL(lanczos_update_kernel, dim3(d.wgs), dim3(kThreads), 0, st, A.n, w, u, u_prev, j, d.beta,
                       d.part_a, d.wgs, d.alpha, d.part_b);
    return hipGetLastError();
}

hipError_t launch_lanczos_beta(const LanczosDev& d, int j, hipStream_t st) {
    hipLaunchKernelGGL(lanczos_beta_kernel, dim3(1), dim3(kThreads), 0, st, d.part_b, d.wgs, d.beta, j);
    return hipGetLastError();
}

}  // namespace ld
