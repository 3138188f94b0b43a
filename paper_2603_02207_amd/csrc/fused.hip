// Several Newton steps per launch on 2-D five-point stencils.
//
// For a matrix stored as constant diagonals at offsets -D, -1, 0, 1, D, the
// row r = y D + x couples only to its neighbours in line y and to lines y +- 1.
// A wave owns a strip: 64 consecutive positions x of every line (one lane
// each) and one 16-byte chunk of columns, and walks the lines in order.  Each
// line is loaded once; level t (t = 1..LV) then computes line y - t of the
// vector after t steps from three lines of level t - 1, all in registers: the
// neighbours x +- 1 come from the adjacent lanes (DPP), the lines above and
// below from the wave's own ring of three lines per level.  There is no LDS,
// no barrier and no exchange between waves.  Each level loses one valid lane
// on either side, so the strip's inner 64 - 2 LV positions are written, and
// the LV lines before and after a wave's own lines are walked too.
//
// The single-step kernels move the block through the memory system once per
// step (28.5-36 us at 20 FP32 columns and 1024^2 points, 6 TB/s from the
// Infinity Cache); here it moves once per LV steps and the vector ALUs become
// the bound: about 35 instructions per step and chunk, a third of them on the
// lanes and lines two waves both walk (the table at fused_levels).  By counters
// they are busy for 73% of a launch of six sketch steps and 55% of one of three
// quadratic-form steps (1024^2 points, 20 FP32 columns; 41% of four adaptive
// steps at 2048^2); the rest is latency at 2.1 to 2.4 waves a SIMD in the mean
// (3.9 at the start: they end at different times).  To that end alpha is folded into the diagonals' values and alpha*centre - beta into
// one coefficient (both formed in FP64): five products per element, in the
// order of the offsets, where the single steps take seven.  Two positions per
// lane measured slower (17.9 against 15.6 us per step at four levels): half
// the waves, too few to cover the loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <type_traits>

#include "kernels.h"

namespace ld {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

template <typename T, int V>
struct alignas(sizeof(T) * V) Chunk {
    T v[V];
};

// the value of the lane before (wave_shr:1) or after (wave_shl:1); zero past the wave's ends
template <int CTRL>
__device__ __forceinline__ float lane_shift(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int kFromBefore = 0x138, kFromAfter = 0x130;

// x with the sign bit of `bit31`
__device__ __forceinline__ float with_sign(float x, unsigned bit31) {
    return __uint_as_float((bit31 & 0x80000000u) ^ __float_as_uint(x));
}
__device__ __forceinline__ double with_sign(double x, unsigned bit31) {
    return __hiloint2double((int)((bit31 & 0x80000000u) ^ (unsigned)__double2hiint(x)), __double2loint(x));
}

template <typename T>
struct FusedDev {
    int n, D, lines;
    int rows_per_chunk;        // lines of one wave's own
    int strips, nq, items;     // strips x line chunks x column chunks
    int width;                 // positions of a line a strip writes
    const T* win;
    long long win_cs;          // elements between column chunks of the input block
    int win_rs;                // elements between rows of the input block
    T* wout;
    long long wout_cs;
    int wout_rs;
    const uint16_t* pres;
    const uint8_t* planes;     // SIGNS: byte planes of the sign words
    int gcol;                  // SIGNS: global column of the block's first column
    const T* vsrc;             // VECS: V, chunk-blocked as the output
    long long vsrc_cs;
    int vsrc_rs;
    double* part;              // DOT: [slot][strip x line chunk][part_ld]
    long long slot_stride;
    int part_ld, bcols;
    int store, nt_out;
    const T* pin;              // ACC: the accumulator, laid out as the output (win and wout too)
    T* pout;
    const uint64_t* active;    // ACC: the columns that accumulate level t's term, bit c of active[t]
    const int* run;            // ACC: when non-null, the launch does nothing unless *run != 0
    T init;                    // INIT: level 0 = init * S (or V); ACC: the accumulator = init * the input
    T c[5];                    // alpha * diagonal value (the centre's is in mid)
    T mid[kFusedMax], nbeta[kFusedMax], dj[kFusedMax];   // alpha * centre - beta, -beta
};

// acc[e] += c * x[e] of the lane before / after (zero past the wave's ends).  The
// compiler does not put the lane shift into the FP32 product itself (a third of
// a step's instructions otherwise); the no-op covers the two wait states
// between a vector write and a DPP read of it.
template <int CTRL>
__device__ __forceinline__ void add_shifted(float (&acc)[4], const float (&x)[4], float c) {
    if constexpr (CTRL == kFromBefore)
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %4, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %1, %5, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %2, %6, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %3, %7, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
            : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(c));
    else
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %4, %8 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %1, %5, %8 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %2, %6, %8 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
            "v_fmac_f32_dpp %3, %7, %8 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
            : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2]), "+&v"(acc[3])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(c));
}
template <int CTRL>
__device__ __forceinline__ void add_shifted(double (&acc)[2], const double (&x)[2], double c) {
#pragma unroll
    for (int e = 0; e < 2; ++e) acc[e] = fma(c, lane_shift<CTRL>(x[e]), acc[e]);
}

template <typename T, int VEC, int KIND, int LV, bool INIT>
__global__ __launch_bounds__(kThreads) void fused_kernel(const FusedDev<T> a) {
    static_assert(KIND == STEP_HORNER_SIGNS || KIND == STEP_HORNER_VEC || KIND == STEP_DOT_SQ || KIND == STEP_ACC_NORM,
                  "fused kinds");
    constexpr bool kSigns = KIND == STEP_HORNER_SIGNS, kVec = KIND == STEP_HORNER_VEC, kDot = KIND == STEP_DOT_SQ;
    constexpr bool kAcc = KIND == STEP_ACC_NORM, kSum = kDot || kAcc;
    constexpr bool kFirst = kDot && INIT;   // the sums of the input block too
    constexpr bool kReadAcc = kAcc && !INIT;
    if (kAcc && ((a.run && *a.run == 0) || a.active[0] == 0)) return;
    constexpr bool kReadIn = !(INIT && (kSigns || kVec));
    using P = Chunk<T, VEC>;
    const int lane = threadIdx.x & 63;
    // XCD x (= blockIdx % 8) takes a contiguous band of workgroups
    const int xcd = blockIdx.x % kXcds, per = gridDim.x / kXcds, rem = gridDim.x % kXcds;
    const int wg = xcd * per + (xcd < rem ? xcd : rem) + blockIdx.x / kXcds;
    const int item = __builtin_amdgcn_readfirstlane(wg * kWaves + (int)(threadIdx.x >> 6));
    if (item >= a.items) return;   // whole waves
    const int q = item % a.nq, sc = item / a.nq;
    const int strip = sc % a.strips, yc = sc / a.strips;
    const int x = strip * a.width + lane - LV;
    const bool own = lane >= LV && lane < LV + a.width && x < a.D;
    const int y0 = yc * a.rows_per_chunk, ny = min(a.rows_per_chunk, a.lines - y0);
    // line y0 - LV + k is loaded in iteration k; its row of this lane is r0 + k D
    const int r0 = (y0 - LV) * a.D + x;
    const T* const win = a.win + (size_t)q * a.win_cs;
    const T* const vsrc = kVec ? a.vsrc + (size_t)q * a.vsrc_cs : nullptr;
    T* const wout = a.wout + (size_t)q * a.wout_cs;
    const int g = a.gcol + q * VEC;
    const uint8_t* const plane = kSigns ? a.planes + (size_t)((g >> 3) & 7) * a.n : nullptr;
    const int pshift = g & 7;

    P ring[LV][3];                 // three lines of levels 0 .. LV-1
    unsigned meta[LV + 1];         // line of level t: presence bits, and the chunk's sign bits at the top
    P vline[kVec ? LV + 1 : 1];    // VECS: V's line of level t
    unsigned full = 0;             // bit t: every lane of level t's line has all five entries
    P accl[kAcc ? LV + 1 : 1];     // ACC: the accumulator's line of level t
    unsigned on[kAcc ? LV : 1];    // ACC: the chunk's columns that take level t + 1's term
    double s0[VEC], s1[kDot ? LV : 1][VEC], s2[kSum ? LV : 1][VEC];
    const long long pofs = (long long)q * a.wout_cs;
#pragma unroll
    for (int t = 0; t < (kAcc ? LV : 1); ++t) on[t] = kAcc ? (unsigned)(a.active[t] >> (q * VEC)) : 0u;   // q*VEC < 64
#pragma unroll
    for (int t = 0; t <= LV; ++t) meta[t] = 0;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        s0[e] = 0.0;
#pragma unroll
        for (int t = 0; t < (kDot ? LV : 1); ++t) s1[t][e] = 0.0;
#pragma unroll
        for (int t = 0; t < (kSum ? LV : 1); ++t) s2[t][e] = 0.0;
#pragma unroll
        for (int t = 0; t < (kAcc ? LV + 1 : 1); ++t) accl[t].v[e] = T(0);
#pragma unroll
        for (int t = 0; t < LV; ++t) ring[t][0].v[e] = ring[t][1].v[e] = ring[t][2].v[e] = T(0);
#pragma unroll
        for (int t = 0; t < (kVec ? LV + 1 : 1); ++t) vline[t].v[e] = T(0);
    }

    // three lines in flight
    P wf[kReadIn ? 3 : 1], vf[kVec ? 3 : 1], af[kReadAcc ? 3 : 1];
    unsigned pm[3], pb[3];
    const int iters = ny + 2 * LV;
    auto fetch = [&](int k, int s) __attribute__((always_inline)) {
        const int r = r0 + k * a.D;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (kReadIn) wf[kReadIn ? s : 0].v[e] = T(0);
            if (kVec) vf[kVec ? s : 0].v[e] = T(0);
            if (kReadAcc) af[kReadAcc ? s : 0].v[e] = T(0);
        }
        pm[s] = pb[s] = 0;
        if (k < iters && (unsigned)r < (unsigned)a.n) {
            if (kReadIn) wf[kReadIn ? s : 0] = *reinterpret_cast<const P*>(win + (size_t)r * a.win_rs);
            if (kVec) vf[kVec ? s : 0] = *reinterpret_cast<const P*>(vsrc + (size_t)r * a.vsrc_rs);
            if (kReadAcc) af[kReadAcc ? s : 0] = *reinterpret_cast<const P*>(a.pin + pofs + (size_t)r * a.wout_rs);
            pm[s] = a.pres[r];
            if (kSigns) pb[s] = plane[r];
        }
    };
    fetch(0, 0);
    fetch(1, 1);
    fetch(2, 2);

    auto iteration = [&](int k, auto slot) __attribute__((always_inline)) {
        constexpr int S = decltype(slot)::value, S1 = (S + 2) % 3, S2 = (S + 1) % 3;   // line k, k-1, k-2
#pragma unroll
        for (int t = LV; t >= 1; --t) {
            meta[t] = meta[t - 1];
            if (kVec) vline[kVec ? t : 0] = vline[kVec ? t - 1 : 0];
            if (kAcc) accl[kAcc ? t : 0] = accl[kAcc ? t - 1 : 0];   // level t - 1's line of the iteration before
        }
        meta[0] = pm[S];
        if (kSigns) meta[0] |= (pb[S] >> pshift) << (32 - VEC);
        full = (full << 1) | (__ballot((pm[S] & 31u) != 31u) == 0 ? 1u : 0u);
        if (kVec) vline[0] = vf[kVec ? S : 0];
        if (kReadIn) ring[0][S] = wf[kReadIn ? S : 0];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (INIT && kSigns) ring[0][S].v[e] = with_sign(a.init, meta[0] << (VEC - 1 - e));
            if (INIT && kVec) ring[0][S].v[e] = a.init * vline[0].v[e];
            if (kAcc) accl[0].v[e] = INIT ? a.init * wf[kReadIn ? S : 0].v[e] : af[kReadAcc ? S : 0].v[e];
        }
        fetch(k + 3, S);
#pragma unroll
        for (int t = 1; t <= LV; ++t) {
            if (k < 2 * t) break;   // level t starts at line y0 - (LV - t) (the same for the whole wave)
            const P &up = ring[t - 1][S2], &mid = ring[t - 1][S1], &dn = ring[t - 1][S];
            P o;
            if ((full >> t) & 1u) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) o.v[e] = a.c[0] * up.v[e];
                add_shifted<kFromBefore>(o.v, mid.v, a.c[1]);
#pragma unroll
                for (int e = 0; e < VEC; ++e) o.v[e] = fma(a.mid[t - 1], mid.v[e], o.v[e]);
                add_shifted<kFromAfter>(o.v, mid.v, a.c[3]);
#pragma unroll
                for (int e = 0; e < VEC; ++e) o.v[e] = fma(a.c[4], dn.v[e], o.v[e]);
            } else {   // an absent entry takes no part, whatever its neighbour holds
                const unsigned m = meta[t];
                const T cm = (m & 4u) ? a.mid[t - 1] : a.nbeta[t - 1];
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const T lf = lane_shift<kFromBefore>(mid.v[e]), rt = lane_shift<kFromAfter>(mid.v[e]);
                    T s = a.c[0] * ((m & 1u) ? up.v[e] : T(0));
                    s = fma(a.c[1], (m & 2u) ? lf : T(0), s);
                    s = fma(cm, mid.v[e], s);
                    s = fma(a.c[3], (m & 8u) ? rt : T(0), s);
                    o.v[e] = fma(a.c[4], (m & 16u) ? dn.v[e] : T(0), s);
                }
            }
            // last: one rounding at the term's size
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if (kSigns) o.v[e] += with_sign(a.dj[t - 1], meta[t] << (VEC - 1 - e));
                if (kVec) o.v[e] = fma(a.dj[t - 1], vline[kVec ? t : 0].v[e], o.v[e]);
                if (kAcc && ((on[kAcc ? t - 1 : 0] >> e) & 1u))
                    accl[kAcc ? t : 0].v[e] = fma(a.dj[t - 1], o.v[e], accl[kAcc ? t : 0].v[e]);
            }
            const int ly = k - t - LV;   // the line's index among the wave's own
            if (kSum && ly >= 0 && ly < ny && own) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const double wd = (double)mid.v[e], od = (double)o.v[e];
                    if (kFirst && t == 1) s0[e] = fma(wd, wd, s0[e]);
                    if (kDot) s1[kDot ? t - 1 : 0][e] = fma(wd, od, s1[kDot ? t - 1 : 0][e]);
                    s2[kSum ? t - 1 : 0][e] = fma(od, od, s2[kSum ? t - 1 : 0][e]);
                }
            }
            if (t < LV) {
                ring[t < LV ? t : 0][S] = o;
            } else if (a.store) {
                const int r = r0 + (k - LV) * a.D;
                if (own && (unsigned)r < (unsigned)a.n) {
                    T* const dst = wout + (size_t)r * a.wout_rs;
                    if (a.nt_out) {
                        typedef T vt __attribute__((ext_vector_type(VEC)));
                        vt v;
#pragma unroll
                        for (int e = 0; e < VEC; ++e) v[e] = o.v[e];
                        __builtin_nontemporal_store(v, reinterpret_cast<vt*>(dst));
                    } else {
                        *reinterpret_cast<P*>(dst) = o;
                    }
                    if (kAcc) *reinterpret_cast<P*>(a.pout + pofs + (size_t)r * a.wout_rs) = accl[kAcc ? LV : 0];
                }
            }
        }
    };
    int k = 0;
    for (; k + 3 <= iters; k += 3) {
        iteration(k, std::integral_constant<int, 0>{});
        iteration(k + 1, std::integral_constant<int, 1>{});
        iteration(k + 2, std::integral_constant<int, 2>{});
    }
    if (k < iters) iteration(k, std::integral_constant<int, 0>{});
    if (k + 1 < iters) iteration(k + 1, std::integral_constant<int, 1>{});

    if constexpr (kSum) {   // butterfly over the wave, lane 0 writes the wave's partial row
        const size_t at = (size_t)sc * a.part_ld + q * VEC;
        auto total = [&](double v, int slot, int e) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 32; h >= 1; h >>= 1) v += __shfl_xor(v, h, 64);
            if (lane == 0 && q * VEC + e < a.bcols) a.part[(size_t)slot * a.slot_stride + at + e] = v;
        };
        constexpr int base = kFirst ? 1 : 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (kFirst) total(s0[e], 0, e);
#pragma unroll
            for (int t = 0; t < LV; ++t) {
                if (kDot) total(s1[kDot ? t : 0][e], base + 2 * t, e);
                total(s2[t][e], kDot ? base + 2 * t + 1 : t, e);
            }
        }
    }
}

template <typename T, int VEC, int KIND, int LV>
hipError_t launch_fused_lv(const FusedDev<T>& d, bool init, hipStream_t st) {
    const int nwg = (d.items + kWaves - 1) / kWaves;
    if (init)
        hipLaunchKernelGGL((fused_kernel<T, VEC, KIND, LV, true>), dim3(nwg), dim3(kThreads), 0, st, d);
    else
        hipLaunchKernelGGL((fused_kernel<T, VEC, KIND, LV, false>), dim3(nwg), dim3(kThreads), 0, st, d);
    return hipGetLastError();
}

template <typename T, int KIND, int LV = 1>
hipError_t launch_fused_k(const FusedDev<T>& d, int levels, bool init, hipStream_t st) {
    if constexpr (LV <= fused_levels(KIND, sizeof(T) == 8)) {
        if (levels == LV) return launch_fused_lv<T, 16 / (int)sizeof(T), KIND, LV>(d, init, st);
        return launch_fused_k<T, KIND, LV + 1>(d, levels, init, st);
    } else {
        return hipErrorInvalidValue;
    }
}

template <typename T>
hipError_t launch_fused_t(const FusedArgs& f, hipStream_t st) {
    constexpr int VEC = 16 / (int)sizeof(T);
    FusedDev<T> d{};
    d.n = f.n;
    d.D = f.D;
    d.lines = (int)(((long long)f.n + f.D - 1) / f.D);
    const FusedGrid gr = fused_grid(f.kind, f.n, f.D, f.bcols, (int)sizeof(T), f.grid_levels, f.max_parts);
    d.rows_per_chunk = gr.rows;
    d.strips = gr.strips;
    d.width = 64 - 2 * f.grid_levels;
    d.nq = (f.bcols + VEC - 1) / VEC;
    d.items = gr.parts * d.nq;
    d.win = (const T*)f.win;
    d.win_cs = f.win_cs;
    d.win_rs = f.win_rs;
    d.wout = (T*)f.wout;
    d.wout_cs = f.wout_cs;
    d.wout_rs = f.wout_rs;
    d.pres = f.pres;
    d.planes = f.planes;
    d.gcol = f.gcol;
    d.vsrc = (const T*)f.vsrc;
    d.vsrc_cs = f.vsrc_cs;
    d.vsrc_rs = f.vsrc_rs;
    d.part = f.part;
    d.slot_stride = f.slot_stride;
    d.part_ld = f.part_ld;
    d.bcols = f.bcols;
    d.store = f.wout != nullptr;
    d.nt_out = f.nt_out;
    d.pin = (const T*)f.pin;
    d.pout = (T*)f.pout;
    d.active = f.active;
    d.run = f.run;
    d.init = (T)f.init_scale;
    for (int q = 0; q < 5; ++q) d.c[q] = (T)f.off[q];
    for (int t = 0; t < f.levels; ++t) {
        d.mid[t] = (T)f.mid[t];
        d.nbeta[t] = (T)f.nbeta[t];
        d.dj[t] = (T)f.dj[t];
    }
    switch (f.kind) {
        case STEP_HORNER_SIGNS: return launch_fused_k<T, STEP_HORNER_SIGNS>(d, f.levels, f.init, st);
        case STEP_HORNER_VEC: return launch_fused_k<T, STEP_HORNER_VEC>(d, f.levels, f.init, st);
        case STEP_DOT_SQ: return launch_fused_k<T, STEP_DOT_SQ>(d, f.levels, f.init, st);
        case STEP_ACC_NORM:
            if (!f.active || !f.pout || !f.wout) return hipErrorInvalidValue;
            return launch_fused_k<T, STEP_ACC_NORM>(d, f.levels, f.init, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

FusedGrid fused_grid(int kind, int n, int D, int bcols, int elem, int levels, int max_parts) {
    const int vec = 16 / elem, nq = (bcols + vec - 1) / vec;
    const int lines = (int)(((long long)n + D - 1) / D), width = 64 - 2 * levels;
    FusedGrid g{};
    g.strips = (D + width - 1) / width;
    int want = std::max(1, kFusedWaves / (g.strips * nq));   // line chunks that fill the device
    if (max_parts > 0) want = std::min(want, std::max(1, max_parts / g.strips));
    const int idle = std::max(1, fused_idle_waves(kind) / (g.strips * nq));
    g.rows = std::max((lines + want - 1) / want,
                      std::min({lines, kFusedMinLines, std::max(2, (lines + idle - 1) / idle)}));
    g.parts = g.strips * ((lines + g.rows - 1) / g.rows);
    return g;
}

hipError_t launch_fused(bool f64, const FusedArgs& f, hipStream_t st) {
    if (f.levels < 1 || f.levels > f.grid_levels || f.grid_levels > kFusedMax || f.bcols < 1 || f.D < 2 || !f.pres) return hipErrorInvalidValue;
    if ((long long)f.n + (long long)(2 * kFusedMax + 4) * f.D >= INT_MAX) return hipErrorInvalidValue;
    return f64 ? launch_fused_t<double>(f, st) : launch_fused_t<float>(f, st);
}

}  // namespace ld
