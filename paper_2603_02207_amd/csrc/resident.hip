// Whole recurrences of a small matrix in one launch.
//
// The columns of a block never interact, so a workgroup can run all the steps
// of one 16-byte column chunk by itself.  When the matrix (16-bit columns and
// values) and the chunk's current vector fit a CU's LDS, a step is then a pass
// over the rows from LDS and two workgroup barriers, where a launch per step
// costs 4-6 us whatever it does.  Each thread keeps its rows' new values, signs
// or V in registers.  Rows are summed in CSR order, products as in the
// single-step kernels.  Measured on gfx950, 32^2 grid, FP32: 40 sketch steps over
// 10 columns 220 -> 55 us, 20 quadratic-form steps over 20 columns 160 -> 75 us
// (launches and gaps against one launch), the estimate 553 -> 358 us.  Larger
// matrices gain less, since one workgroup walks all rows of a chunk, and never
// lose: FP32 estimates of degree 40 and 60 queries against single steps, 40^2
// grid 559 -> 453 us, 50^2 556 -> 500, 58^2 559 -> 545; tridiagonal, 2500 rows
// 533 -> 437, 4090 rows 542 -> 485.
// More than four rows a thread do not fit its 128 registers: the column sums
// spill from the fifth row, all kinds at eight, to scratch that the runtime may
// have to allocate; such matrices keep single steps.
//
// Bound by LDS latency (a row's gathers) and the barriers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <set>

#include "kernels.h"

namespace ld {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

template <typename T, int V>
struct alignas(sizeof(T) * V) Chunk {
    T v[V];
};

template <typename T>
struct ResidentDev {
    int n, nnz;
    const int *row_ptr, *col_idx;
    const T* val;
    int cols, steps;
    const T* src;              // SIGNS: null; else V or X: element (r, c) at r * src_ld + c (+ block offset)
    int src_ld, src_vec;       // src_vec: rows are whole aligned vectors
    T* out;                    // SIGNS, VEC, ADAPT: as src
    int out_ld, out_vec;
    const uint64_t* mask;      // SIGNS
    int gcol;
    double* part;              // DOT: [slot][kWaves][part_ld]
    long long slot_stride;
    int part_ld;
    double tol;                // ADAPT
    int* deg;
    T alpha, init;
    T beta[kResidentSteps];
    double d[kResidentSteps + 1];   // added terms (Horner order) or coefficients (ADAPT)
};

template <typename T, int VEC>
__device__ __forceinline__ Chunk<T, VEC> load_row(const T* p, bool vec, int have) {
    if (vec) return *reinterpret_cast<const Chunk<T, VEC>*>(p);
    Chunk<T, VEC> x;
#pragma unroll
    for (int e = 0; e < VEC; ++e) x.v[e] = e < have ? p[e] : T(0);
    return x;
}

template <typename T, int VEC>
__device__ __forceinline__ void store_row(T* p, const Chunk<T, VEC>& x, bool vec, int have) {
    if (vec) {
        *reinterpret_cast<Chunk<T, VEC>*>(p) = x;
        return;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        if (e < have) p[e] = x.v[e];
}

// The sums of N values (a power of two) over the wave, N + 2 shuffles for N = 8:
// halving the values a lane carries with the lanes it has met, then plain
// exchanges.  Lane l ends with the sum of value wave_slot<N>(l) in v[0].  (A
// butterfly for each value, 48 shuffles a step for 16 waves on one LDS, took
// 4 of the 5.6 us of a quadratic-form step.)
template <int N>
__device__ __forceinline__ int wave_slot(int lane) {
    int slot = 0;
#pragma unroll
    for (int h = 32, k = N / 2; k >= 1; h >>= 1, k >>= 1) slot |= (lane & h) ? k : 0;
    return slot;
}
template <int N>
__device__ __forceinline__ void wave_sums(double (&v)[N], int lane) {
#pragma unroll
    for (int h = 32, k = N / 2; h >= 1; h >>= 1, k >>= 1) {
        if (k >= 1) {
            const bool hi = (lane & h) != 0;
#pragma unroll
            for (int j = 0; j < (k > 0 ? k : 1); ++j) {
                const double send = hi ? v[j] : v[j + k], keep = hi ? v[j + k] : v[j];
                v[j] = keep + __shfl_xor(send, h, 64);
            }
        } else {
            v[0] += __shfl_xor(v[0], h, 64);
        }
    }
}

// RPT rows of a thread: r = threadIdx.x + i * kThreads.
template <typename T, int VEC, int KIND, int RPT>
__global__ __launch_bounds__(kThreads) void resident_kernel(const ResidentDev<T> a) {
    constexpr bool kSigns = KIND == STEP_HORNER_SIGNS, kVec = KIND == STEP_HORNER_VEC;
    constexpr bool kDot = KIND == STEP_DOT_SQ, kAdapt = KIND == STEP_ACC_NORM;
    using P = Chunk<T, VEC>;
    extern __shared__ __align__(16) unsigned char lds[];
    P* const cur = reinterpret_cast<P*>(lds);
    T* const val = reinterpret_cast<T*>(lds + (size_t)a.n * sizeof(P));
    uint16_t* const col = reinterpret_cast<uint16_t*>(val + a.nnz);
    __shared__ double s_norm[kAdapt ? kWaves * VEC : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.x * VEC, have = min(VEC, a.cols - c0);
    for (int k = tid; k < a.nnz; k += kThreads) {
        val[k] = a.val[k];
        col[k] = (uint16_t)a.col_idx[k];
    }
    int beg[RPT], end[RPT];
    unsigned sgn[kSigns ? RPT : 1];
    P keep[kVec || kAdapt ? RPT : 1];   // V of the row; ADAPT: the accumulator
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = tid + i * kThreads;
        beg[i] = end[i] = 0;
        if (r >= a.n) continue;
        beg[i] = a.row_ptr[r];
        end[i] = a.row_ptr[r + 1];
        P x;
        if constexpr (kSigns) {
            sgn[i] = (unsigned)(a.mask[r] >> ((a.gcol + c0) & 63));
#pragma unroll
            for (int e = 0; e < VEC; ++e) x.v[e] = (sgn[i] >> e) & 1u ? -a.init : a.init;
        } else {
            x = load_row<T, VEC>(a.src + (size_t)r * a.src_ld + c0, a.src_vec, have);
            if constexpr (kVec || kAdapt) {
                keep[i] = x;
                if constexpr (kVec)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) x.v[e] = a.init * x.v[e];
            }
        }
        cur[r] = x;
    }
    __syncthreads();

    // ADAPT: |d_m| ||w_m|| against tol, the same in every thread; clears the columns that stop at m
    unsigned active = (1u << have) - 1u;
    auto decide = [&](const double(&sq)[VEC], int m) __attribute__((always_inline)) {
        double v[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[e] = sq[e];
        wave_sums<VEC>(v, lane);
        if ((lane & (64 / VEC - 1)) == 0) s_norm[wave * VEC + wave_slot<VEC>(lane)] = v[0];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            double s = 0.0;
            for (int wv = 0; wv < kWaves; ++wv) s += s_norm[wv * VEC + e];
            const bool on = (active >> e) & 1u;
            if (on && !(fabs(a.d[m]) * sqrt(fmax(s, 0.0)) > a.tol)) {
                active &= ~(1u << e);
                if (tid == 0) a.deg[c0 + e] = m;
            }
        }
        __syncthreads();
    };
    if constexpr (kAdapt) {
        double sq[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) sq[e] = 0.0;
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (tid + i * kThreads < a.n)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const double x = (double)keep[i].v[e];
                    sq[e] = fma(x, x, sq[e]);
                    keep[i].v[e] = a.init * keep[i].v[e];   // P = (d_0 + shift) w_0
                }
        decide(sq, 0);
    }

    P next[RPT];
    for (int j = 0; j < a.steps && (!kAdapt || active); ++j) {
        double s0[VEC], s1[VEC], s2[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s0[e] = s1[e] = s2[e] = 0.0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = tid + i * kThreads;
            if (r >= a.n) continue;
            T acc[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] = T(0);
#pragma unroll 4
            for (int k = beg[i]; k < end[i]; ++k) {
                const P x = cur[col[k]];
                const T v = val[k];
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = fma(v, x.v[e], acc[e]);
            }
            const P w = cur[r];
            P o;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                o.v[e] = a.alpha * acc[e] - a.beta[j] * w.v[e];
                if constexpr (kSigns) o.v[e] = fma((T)a.d[j], (sgn[i] >> e) & 1u ? T(-1) : T(1), o.v[e]);
                if constexpr (kVec) o.v[e] = fma((T)a.d[j], keep[i].v[e], o.v[e]);
                if constexpr (kDot) {
                    if (j == 0) s0[e] += (double)w.v[e] * (double)w.v[e];
                    s1[e] += (double)w.v[e] * (double)o.v[e];
                    s2[e] += (double)o.v[e] * (double)o.v[e];
                }
                if constexpr (kAdapt) {
                    s2[e] += (double)o.v[e] * (double)o.v[e];
                    if ((active >> e) & 1u) keep[i].v[e] = fma((T)a.d[j + 1], o.v[e], keep[i].v[e]);
                }
            }
            next[i] = o;
        }
        __syncthreads();   // every gather of this step is done
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (tid + i * kThreads < a.n) cur[tid + i * kThreads] = next[i];
        if constexpr (kDot) {
            double* const p = a.part + (size_t)wave * a.part_ld + c0;
            if (j == 0) {
                wave_sums<VEC>(s0, lane);
                const int e = wave_slot<VEC>(lane);
                if ((lane & (64 / VEC - 1)) == 0 && e < have) p[e] = s0[0];
            }
            double v[2 * VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                v[e] = s1[e];
                v[VEC + e] = s2[e];
            }
            wave_sums<2 * VEC>(v, lane);
            const int at = wave_slot<2 * VEC>(lane), e = at % VEC;
            if ((lane & (32 / VEC - 1)) == 0 && e < have)
                p[(size_t)(2 * j + 1 + at / VEC) * a.slot_stride + e] = v[0];
        }
        if constexpr (kAdapt)
            decide(s2, j + 1);   // its barriers also publish cur
        else
            __syncthreads();
    }
    if constexpr (kAdapt) {   // columns still active stop at the cap
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if (((active >> e) & 1u) && tid == 0) a.deg[c0 + e] = a.steps;
    }
    if constexpr (!kDot) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = tid + i * kThreads;
            if (r < a.n)
                store_row<T, VEC>(a.out + (size_t)r * a.out_ld + c0, kAdapt ? keep[kVec || kAdapt ? i : 0] : next[i],
                                  a.out_vec, have);
        }
    }
}

// Lets a kernel take more than 64 KB of dynamic LDS (once per kernel and device).
hipError_t allow_lds(const void* fn) {
    static std::mutex mu;
    static std::set<std::pair<int, const void*>> done;
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    std::lock_guard<std::mutex> lock(mu);
    if (done.count({dev, fn})) return hipSuccess;
    if (hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kResidentLds)) return e;
    done.insert({dev, fn});
    return hipSuccess;
}

template <typename T, int KIND>
hipError_t launch_resident_k(const CsrDev& A, const ResidentDev<T>& d, hipStream_t st) {
    constexpr int VEC = 16 / (int)sizeof(T);
    const size_t lds = resident_lds(A.n, A.nnz, (int)sizeof(T));
    const int rpt = (A.n + kThreads - 1) / kThreads;
#define LD_RES(RPT_)                                                                                             \
    {                                                                                                            \
        const auto fn = resident_kernel<T, VEC, KIND, RPT_>;                                                     \
        if (hipError_t e = allow_lds(reinterpret_cast<const void*>(fn))) return e;                               \
        hipLaunchKernelGGL(fn, dim3((d.cols + VEC - 1) / VEC), dim3(kThreads), lds, st, d);                      \
        return hipGetLastError();                                                                                \
    }
    if (rpt <= 1) LD_RES(1)
    if (rpt <= 2) LD_RES(2)
    if (rpt <= 4) LD_RES(4)   // kResidentRows
#undef LD_RES
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_resident_t(const CsrDev& A, const ResidentArgs& f, hipStream_t st) {
    constexpr int VEC = 16 / (int)sizeof(T);
    ResidentDev<T> d{};
    d.n = A.n;
    d.nnz = A.nnz;
    d.row_ptr = A.row_ptr;
    d.col_idx = A.col_idx;
    d.val = (const T*)A.val;
    d.cols = f.cols;
    d.steps = f.steps;
    const auto vec = [](const void* p, int ld) { return (uintptr_t)p % 16 == 0 && ld % VEC == 0; };
    d.src = (const T*)f.src;
    d.src_ld = f.src_ld;
    d.src_vec = vec(f.src, f.src_ld);
    d.out = (T*)f.out;
    d.out_ld = f.out_ld;
    d.out_vec = vec(f.out, f.out_ld);
    d.mask = f.mask;
    d.gcol = f.gcol;
    d.part = f.part;
    d.slot_stride = f.slot_stride;
    d.part_ld = f.part_ld;
    d.tol = f.tol;
    d.deg = f.deg;
    d.alpha = (T)f.alpha;
    d.init = (T)f.init;
    for (int j = 0; j < f.steps; ++j) d.beta[j] = (T)f.beta[j];
    if (f.d)
        for (int j = 0; j < f.steps + (f.kind == STEP_ACC_NORM ? 1 : 0); ++j) d.d[j] = f.d[j];
    switch (f.kind) {
        case STEP_HORNER_SIGNS: return launch_resident_k<T, STEP_HORNER_SIGNS>(A, d, st);
        case STEP_HORNER_VEC: return launch_resident_k<T, STEP_HORNER_VEC>(A, d, st);
        case STEP_DOT_SQ: return launch_resident_k<T, STEP_DOT_SQ>(A, d, st);
        case STEP_ACC_NORM: return launch_resident_k<T, STEP_ACC_NORM>(A, d, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

size_t resident_lds(long long n, long long nnz, int elem) { return (size_t)(n * 16 + nnz * (elem + 2) + 15) / 16 * 16; }

hipError_t launch_resident(bool f64, const CsrDev& A, const ResidentArgs& f, hipStream_t st) {
    if (A.n < 1 || A.n > kResidentRows || f.steps < 1 || f.steps > kResidentSteps || f.cols < 1 ||
        resident_lds(A.n, A.nnz, f64 ? 8 : 4) > (size_t)kResidentLds)
        return hipErrorInvalidValue;
    return f64 ? launch_resident_t<double>(A, f, st) : launch_resident_t<float>(A, f, st);
}

}  // namespace ld
