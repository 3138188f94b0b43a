// Launchers of the gfx950 kernels (kernels.hip).  All launches are
// asynchronous on `stream`; shapes are checked by the caller (api.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ld {

// Kinds of Newton step (one SpMM pass over a block of columns).
enum StepKind : int {
    STEP_HORNER_SIGNS = 0,  // out = alpha*A*in - beta*in + dj*S   (S from the sign mask)
    STEP_HORNER_VEC = 1,    // out = alpha*A*in - beta*in + dj*V   (V in memory)
    STEP_DOT_FWD = 2,       // out = alpha*A*in - beta*in; <X,out> (and <X,in> if first)
    STEP_DOT_SQ = 3,        // out = alpha*A*in - beta*in; <in,out>, <out,out> (and <in,in>)
    STEP_PLAIN = 4,         // out = alpha*A*in - beta*in
    STEP_PLAIN_ACC = 5,     // PLAIN, and acc[r, c] += dj*out[r, c] for columns c < acc_cols
    STEP_ACC_NORM = 6,      // PLAIN, acc += dj*out on the columns active in *active, <out,out>
};

// A dense n x cols matrix stored as column blocks of width bw: element
// (r, c) lives at (C / bw) * bstride + r * ld + C % bw (in elements), with
// C = c + c0 (c0 selects a column range).  A plain row-major matrix is the
// single-block case.
struct Blk {
    int ld;
    int bw;
    long long bstride;
    int c0;
    __host__ __device__ size_t offset(int c) const {
        const int C = c + c0;
        return (size_t)(C / bw) * (size_t)bstride + (size_t)(C % bw);
    }
    static Blk plain(int ld, int c0 = 0) { return Blk{ld, 1 << 30, 0, c0}; }
    Blk shifted(int dc) const { return Blk{ld, bw, bstride, c0 + dc}; }
};

struct CsrDev {
    int n;
    int nnz;
    const int* row_ptr;
    const int* col_idx;
    const void* val;
};

constexpr int kMaxDiag = 9;
constexpr int kXcds = 8;     // XCDs of the MI355X; workgroup w runs on XCD w % 8      // diagonals of the diagonal storage (9-point stencils, 7-point 3-D)

// Geometry of a Newton step launch over columns [c0, c0+bcols) of row-major
// blocks with leading dimension ld (elements).
struct StepArgs {
    int kind;
    bool first;
    const void* win;
    void* wout;
    int ld, c0, bcols;
    int gshift;                // global column = local column + gshift
    double alpha, beta, dj;
    const void* vsrc;          // HORNER_VEC: V;  DOT_FWD: X
    int ldv;
    const uint64_t* mask;      // HORNER_SIGNS: one word of sign bits per row
    // HORNER_SIGNS on the diagonal storage, when non-null: the same bits as
    // eight byte planes (plane p, n bytes: byte p of every row's word), so a
    // step reads one byte per row and 16-byte chunk instead of the word
    const uint8_t* planes = nullptr;
    double* ps0;               // partial sums [nwg][part_ld], may be null
    double* ps1;
    double* ps2;
    int part_ld;
    // Rows with more than kLongRow entries, when listed here, are skipped by the
    // row-group kernel and done by a launch of their own (partial rows after the
    // regular ones: kLongWgs of them).
    const int* long_rows;      // device list of long rows (ascending), or null
    const int* long_count;     // device count of the list
    void* acc;                 // PLAIN_ACC / ACC_NORM: row-major accumulator (column c of the step = column c)
    int ldacc, acc_cols;
    const uint64_t* active;    // ACC_NORM: device word, bit (c - c0) set = column c still accumulates
    // Diagonal storage of A (dia_nd > 0): row r holds dia[r*dia_nd + q] at
    // column r + dia_off[q] (offsets ascending; 0 where absent); replaces the
    // CSR arrays in the gather.
    const void* dia;
    int dia_nd;
    int dia_off[kMaxDiag];
    // every diagonal one constant (dia_pres non-null): row r holds dia_cval[q]
    // on diagonal q when bit q of dia_pres[r] is set; dia is not read
    const uint16_t* dia_pres;
    double dia_cval[kMaxDiag];
    // tile order: 0 = XCD x (blockIdx % 8) walks the x-th contiguous band of
    // row tiles (stencil neighbours stay in that XCD's L2); 1 = workgroup w
    // takes tiles w, w + grid, ... (spreads each tile's neighbours over the
    // XCDs; faster once the blocks stream from HBM)
    int interleave;
    int scattered = 0;   // most entries lie far from the diagonal (CSR slices)
    // with interleave = 0: > 0 cuts the bands into chunks of about this many
    // rows, chunk c going to XCD c % 8 (each XCD walks its chunks in order);
    // 0 = one contiguous band per XCD
    int chunk_rows;
    // 1: the output block is written with non-temporal (streaming) stores
    int nt_out;
    // when non-null: set to the number of launches over consecutive row
    // ranges the step took (1 but for streaming steps with column sums)
    int* ranges_out = nullptr;
};

constexpr int kLongRow = 64;     // entries above which a row is "long"
constexpr int kLongWgs = 1024;   // workgroups of the long-row launch

// Deterministic list of the rows with more than kLongRow entries:
// list[0..count) ascending, *count on the device.  tmp: >= n/256 + 2 ints.
hipError_t launch_long_rows(const CsrDev& A, int* tmp, int* list, int* count, hipStream_t st);

// Widest column range of one launch (a row group spans at most one wave).
int step_max_cols(bool f64, const StepArgs& s);
// Partial rows a column-sum launch writes (one per workgroup), at most: for
// 16-byte aligned blocks of at most bcols columns, and for any layout.
int step_num_wg_bound(int n, int bcols, int elem_bytes);
int step_num_wg_any(int n);
// Entries of the rows a wave of the row-group CSR kernel takes in one pass, over
// those it can stage in LDS (the row's columns on lpr lanes).
double step_staging(long long n, long long nnz, int lpr);
// Row tiles of a CSR launch with lpr lanes a row.
int step_tiles(int n, int lpr);
// Rows of one tile of the column-sum kinds over bcols columns of 16-byte aligned blocks.
int step_tile_rows(int bcols, int elem_bytes);

// *nwg_out (may be null): workgroup partial rows the launch wrote (dot kinds:
// the grid, which is the number of resident workgroups or less, plus the
// long-row launch's kLongWgs).
hipError_t launch_step(bool f64, const CsrDev& A, const StepArgs& s, hipStream_t st, int* nwg_out = nullptr);

// Several Newton steps per launch on a constant five-point stencil (fused.hip; at
// least kFusedMinWidth rows a line):
// diagonals at offsets -D, -1, 0, 1, D (in that order in off; bit q of pres[r] =
// row r stores diagonal q).  Level t = 0..levels-1 takes w -> alpha*A*w -
// beta_t*w (+ dj[t]*S or + dj[t]*V), off = alpha times the diagonals' values,
// mid[t] = off[2] - beta_t.  Element (r, c) of a block sits at
// (c / VEC)*cs + r*rs + c % VEC, VEC the elements of 16 bytes: row-major rows
// (cs = VEC, rs = ld) or 16-byte column chunks one after another (cs = n*VEC,
// rs = VEC).
//   STEP_HORNER_SIGNS: S from the byte planes of its sign words (gcol = global
//                      column of the block's first column); with init the input
//                      is init_scale*S itself
//   STEP_HORNER_VEC:   V in vsrc; with init the input is init_scale*V
//   STEP_DOT_SQ:       level t writes <in,out>, <out,out> of its step to slots
//                      2t, 2t+1 of part ([slot][partial row][part_ld]); with
//                      init slot 0 takes <in,in> and the others move up by one.
//                      wout null: the last vector is not written.
//   STEP_ACC_NORM:     level t adds dj[t]*w to the accumulator on the columns of
//                      active[t] (device words) and writes <out,out> to slot t;
//                      pin to pout, laid out as the output; with init the
//                      accumulator starts as init_scale*input.  run non-null: the
//                      launch does nothing unless *run (device) is nonzero.
//
// Every launch of a phase takes the grid of grid_levels (>= levels), so that all
// write the same partial rows.
constexpr int kFusedMax = 6;          // most levels of one launch
constexpr int kFusedMinWidth = 128;   // shortest lines taken
constexpr int kFusedWaves = 4096;     // waves a launch aims at: 4 per SIMD
constexpr int kFusedMinLines = 16;    // fewest lines of a wave (each walks 2*levels more), unless
                                      // so many leave most of the device idle (fused_idle_waves)

// Levels of one launch.  Measured on gfx950, us per step (1024^2 points; 20
// FP32 / 10 FP64 columns), against the single-step kernels:
//            levels 1     2     3     4     5     6    single step
//   SIGNS F32    29.4  15.8  12.3  12.8  12.5  11.6    31
//         F64    28.8  15.4  11.5  11.2  11.0  10.7    36
//   VEC   F32    42.6  23.3  17.0  14.2  15.6  16.1    39
//         F64    41.8  22.9  16.3  13.1  13.3  13.7    39
//   SQ    F32    30.6  18.4  15.4  20.0  20.3  20.7    35
//         F64    28.9  16.4  12.1  11.6  14.0  14.8    35
// More levels move fewer bytes per step but walk more lines and lanes twice;
// the column sums (16 registers a level) drop the waves per SIMD from 4 to 3
// above 3 levels in FP32, 4 in FP64.
// ACC_NORM, whole adaptive estimates in ms: FP32, 2048^2, 32 queries of about 49
// steps 14.2 with 3 levels, 11.7 with 4, 11.0 with 5 (30.0 one step at a time);
// 1024^2, 16 queries of 2 to 11 steps 1.30 with 4, 1.43 with 5, 1.46 with 6: 4,
// since columns stop inside a launch and more levels repeat more.
constexpr int fused_levels(int kind, bool f64) {
    return kind == STEP_HORNER_SIGNS ? 6 : kind == STEP_HORNER_VEC || kind == STEP_ACC_NORM ? 4 : f64 ? 4 : 3;
}
// Waves below which a wave takes fewer than kFusedMinLines lines, down to two: the
// device is then mostly idle, a launch lasts as long as one wave's walk, and the
// lines walked twice cost nothing.  Measured (us per step; 16, 8, 4, 2 lines, single
// steps): sketch of 10 FP32 columns, 128 x 62 points 4.57, 3.10, 2.37, 1.95, 3.44;
// quadratic forms of 20 columns 7.27, 5.38, 4.52, 3.92, 5.86; log(A) V, 60 steps,
// one column, 150^2 350, 259, 220, 196, 316 us.  Near a full device two lines cost
// more than eight (350^2, quadratic forms of 40 FP32 columns: 9.1, 8.6 at 4 to 8).
// The adaptive launches' sums are reduced after every one of them, so more waves
// cost more there (20000 x 8 points, one column: 569 us at 8 lines, 618 at two).
constexpr int fused_idle_waves(int kind) { return kind == STEP_ACC_NORM ? 1024 : 2048; }
struct FusedArgs {
    int kind, levels, grid_levels;
    bool init;
    int n, D, bcols;
    const void* win;
    long long win_cs;
    int win_rs;
    void* wout;
    long long wout_cs;
    int wout_rs;
    const uint16_t* pres;
    double off[5];                    // alpha * diagonal value
    const uint8_t* planes;
    int gcol;
    const void* vsrc;
    long long vsrc_cs;
    int vsrc_rs;
    double* part;
    long long slot_stride;
    int part_ld;
    int max_parts;                    // most partial rows (0: no limit)
    int nt_out;
    const void* pin;
    void* pout;
    const uint64_t* active;
    const int* run;
    double init_scale;
    double mid[kFusedMax], nbeta[kFusedMax], dj[kFusedMax];   // off[2] - beta, -beta
};
struct FusedGrid {
    int strips, rows, parts;          // strips of a line, lines of a wave, partial rows
};
FusedGrid fused_grid(int kind, int n, int D, int bcols, int elem, int levels, int max_parts);
hipError_t launch_fused(bool f64, const FusedArgs& f, hipStream_t st);

// Whole recurrences of a matrix whose CSR arrays and one 16-byte column chunk fit
// a CU's LDS (resident.hip): `steps` steps w -> alpha*A*w - beta[j]*w (+ dj*S or
// + dj*V, d[j] in step order) of every chunk of a row-major block of `cols`
// columns, one workgroup per chunk.
//   STEP_HORNER_SIGNS / _VEC: from init*S / init*V (V = src) to out
//   STEP_DOT_SQ:   from src; step j's <in,out>, <out,out> to slots 2j+1, 2j+2 of
//                  part, the first <in,in> to slot 0: kResidentParts partial rows
//   STEP_ACC_NORM: Alg. 2's loop on the columns of src: out = init*v + sum_{m>=1}
//                  d[m]*w_m, each column to the first m with |d[m]| ||w_m|| <= tol
//                  (deg[c] = m) or `steps`
constexpr int kResidentSteps = 200;
constexpr int kResidentRows = 4096;       // four of each of a workgroup's 1024 threads
constexpr int kResidentParts = 16;
constexpr int kResidentLds = 156 << 10;   // of a CU's 160 KB
struct ResidentArgs {
    int kind, cols, steps;
    const void* src;
    int src_ld;
    void* out;
    int out_ld;
    const uint64_t* mask;
    int gcol;
    double* part;
    long long slot_stride;
    int part_ld;
    double tol;
    int* deg;
    double alpha, init;
    const double *beta, *d;   // host
};
size_t resident_lds(long long n, long long nnz, int elem);
hipError_t launch_resident(bool f64, const CsrDev& A, const ResidentArgs& f, hipStream_t st);

// Sign mask of stream `key`: bit c of word r = (probe(r, c) == -1), c < k <= 64.
// With `planes` non-null also its eight byte planes: planes[p*n + r] = byte p
// of word r (8n bytes).
hipError_t launch_sign_mask(int n, int k, uint64_t key, uint64_t* mask, hipStream_t st,
                            uint8_t* planes = nullptr);

// out[r*ld + c] = scale * S[r, c + gshift] for c < k (other columns untouched).
hipError_t launch_fill_signs(bool f64, int n, int k, int ld, int gshift, const uint64_t* mask,
                             double scale, void* out, hipStream_t st);

// out[r, c] = scale * g(key, (c + col0)*n + r + 1), c < k, out column-blocked:
// standard normal entries by Box-Muller (FP64) on the two 32-bit halves of
// SplitMix64 output number (c + col0)*n + r + 1 of the stream key.
hipError_t launch_gauss_fill(bool f64, int n, int k, uint64_t key, int col0, double scale, void* out, Blk bo,
                             hipStream_t st);

// out[r, c] = scale * V[r, c] (row-major, V with ldv, out with ldo), c < ncols.
hipError_t launch_scale_copy(bool f64, int n, int ncols, const void* V, int ldv, double scale,
                             void* out, int ldo, hipStream_t st);

// Row-major V (n x ncols, leading dimension ldv, any alignment) to and from
// 16-byte column chunks one after another (chunk q: n x VEC; columns past ncols
// are zero).
hipError_t launch_pack_chunks(bool f64, int n, int ncols, const void* V, int ldv, void* chunks, hipStream_t st);
hipError_t launch_unpack_chunks(bool f64, int n, int ncols, const void* chunks, void* V, int ldv, hipStream_t st);

// Partial cross products X^T Z per workgroup, FP64: part[wg][i*kz+j],
// cross_num_wg(n) rows.  Z is a second block, or, with zmask (one word per
// row, bit j set = -1), the signs of columns [0, kz); Z is then ignored.
int cross_num_wg(int n);
hipError_t launch_cross(bool f64, int n, const void* X, Blk bx, int kx, const void* Z, Blk bz,
                        int kz, const uint64_t* zmask, double* part, hipStream_t st);

// out[o*out_ld + j] = sum_wg part[o*outer_stride + wg*part_ld + j], j < len
// (Neumaier, fixed order).
hipError_t launch_reduce(const double* part, int nwg, int len, int part_ld, int outer,
                         long long outer_stride, double* out, int out_ld, hipStream_t st);

// G = R^T R for a k x k FP64 Gram (k <= 64, row-major): R (may be null) and
// R^{-1}, both upper triangular; *flag = 0, 1 (non-finite entry) or 2 (pivot
// not positive or below 1e-7 sqrt(G_jj)), R^{-1} zero unless 0.
hipError_t launch_chol_factor(const double* G, int k, double* R, double* Rinv, int* flag,
                              hipStream_t st);

// out[r, j] = (base ? base[r, j] : 0) + (zmask ? sign of bit j of zmask[r] : 0)
//             + sign_m * sum_i Y[r, i] M[i, j],
// M k_y x k_out FP64 (device), j < k_out; Y, base and out column-blocked
// (base may alias out: each element is read before it is written).
hipError_t launch_rowmat(bool f64, int n, const void* Y, Blk by, int ky, const double* M, int kout,
                         double sign_m, const uint64_t* zmask, const void* base, Blk bb,
                         void* out, Blk bo, hipStream_t st);

// CSR structure check: flag[0], flag[1] (device ints, preset to 0) both stay 0
// unless there is a violation.
hipError_t launch_validate_csr(const CsrDev& A, int* flag, hipStream_t st);

// Gershgorin: (min(a_ii - r_i), max(a_ii + r_i)) into out[0..2); part: 2 *
// gersh_num_wg(n) doubles; check: launch_validate_csr's flags (nothing is read
// of a matrix that failed, and the result then means nothing).
int gersh_num_wg(int n);
hipError_t launch_gershgorin(bool f64, const CsrDev& A, const int* check, double* part, double* out, hipStream_t st);

// Gradient sweep step (all blocks n x ld row-major, ncols used; grad FP64):
//   grad[nz(r,c)] (+)= alpha * sum_cols own[r, col] * w[c, col]
//   ADJ_HORNER:  lam_out = alpha*A*lam_in - beta*lam_in + dj*L,  own = lam_in
//   ADJ_PLAIN:   lam_out = alpha*A*lam_in - beta*lam_in,         own = lam_in
//   ADJ_SQUARED: lam_out = alpha*A*lam_in - beta*lam_in + q0*w + q1*(alpha*A*w - beta*w),
//                own = wgt(col) * (lam_in + p1*w), wgt = 1 for col < wsplit, else whi
//   ADJ_PLAIN2 (diagonal storage only): ADJ_PLAIN, and the entry also picks up
//                alpha * sum_cols lam_out[r, col] * w2[c, col] (two steps of the
//                sketch's adjoint per read and write of the gradient)
//   ADJ_SQUARED_SYM (diagonal storage with offsets symmetric about the main
//                diagonal): ADJ_SQUARED's step, and each mirrored pair is summed
//                into the half accumulator of its upper entry: for c > r the
//                slot (r, c) picks up alpha * sum_cols (own[r] w[c] + own[c] w[r]),
//                the diagonal slot alpha * sum_cols own[r] w[r]; slots are
//                grad[r * nh + h] for the h-th non-negative offset (the lower
//                entries have no slot)
enum AdjMode : int { ADJ_HORNER = 0, ADJ_PLAIN = 1, ADJ_SQUARED = 2, ADJ_PLAIN2 = 3, ADJ_SQUARED_SYM = 4 };
struct AdjArgs {
    int mode;
    const void* lam_in;
    void* lam_out;
    const void* w;
    const void* w2;      // ADJ_PLAIN2
    const void* L;
    double* grad;
    int ld, ncols;
    double alpha, beta, dj;
    double q0, q1, p1;   // ADJ_SQUARED coefficients
    int wsplit;          // ADJ_SQUARED column weights: 1 before wsplit, whi after
    double whi;
    bool first;      // grad is overwritten instead of accumulated
    bool last;       // no lam_out needed (only the SDDMM)
    bool nt_out;     // lam_out written with non-temporal (streaming) stores
    double lam_scale = 1.0;   // lam = lam_scale * lam_in (0: a zero block, lam_in not read)
};
hipError_t launch_adjoint(bool f64, const CsrDev& A, const AdjArgs& a, hipStream_t st);

// The same step on the diagonal storage (modes ADJ_PLAIN, ADJ_PLAIN2,
// ADJ_SQUARED, ADJ_SQUARED_SYM): presence bits per row (pres), the values either one per
// diagonal (constant) or dia[r*nd + q]; the gradient at A's CSR positions
// (row_ptr of A).
struct AdjDia {
    int nd;
    int off[kMaxDiag];
    const uint16_t* pres;
    const void* dia;
    bool constant;
    double cval[kMaxDiag];
    int chunk_rows;   // > 0: chunked XCD bands of this many rows (0: contiguous bands)
    int qh0 = 0, nh = 0;   // ADJ_SQUARED_SYM: index of offset 0, number of offsets >= 0
};
hipError_t launch_adjoint_dia(bool f64, const CsrDev& A, const AdjArgs& a, const AdjDia& dg, hipStream_t st);

// Every stored entry of the gradient from the half accumulator of
// ADJ_SQUARED_SYM (half[r * nh + h], nh = dg.nh): g at the CSR position of
// (r, c) = half of the upper entry's pair sum for r != c, the diagonal slot
// for r = c (a mean of mirrored pairs, as launch_symmetrize gives); *flag
// (device int) set to 1 when an entry's mirror is absent.
hipError_t launch_expand_half(const CsrDev& A, const AdjDia& dg, const double* half, double* g, int* flag,
                              hipStream_t st);

// Mean of every mirrored pair g[(r,c)], g[(c,r)] (FP64, CSR positions); *flag
// (device int) set to 1 when some entry has no mirror.
hipError_t launch_symmetrize(const CsrDev& A, double* g, int* flag, hipStream_t st);

// y[i] = (float)x[i], i < len.
hipError_t launch_narrow(long long len, const double* x, float* y, hipStream_t st);

// Row probe (info: device, 64 ints, preset to 0 by the caller): info[0] =
// number of diagonals nd (distinct offsets col - row of 64 sampled rows,
// ascending, in info[1..nd]; -1 if more than kMaxDiag),
// info[kBandInfo + i] = row_ptr[i*n/8], i = 0..8 (entries per XCD band),
// info[kFarInfo] of info[kFarInfo + 1] entries of the sampled rows (at most 16 a
// row) lie more than n/16 rows from the diagonal, and
// at info + kConstInfo nd doubles: each diagonal's value in the first sampled
// row that stores it.  Then the diagonal storage: dia[r*nd + q] =
// A[r, r + info[1+q]] or 0, pres[r] bit q = row r stores diagonal q;
// info[kDiaFlag] = 1 when some stored entry lies on none of the diagonals (the
// storage is then unusable), info[kConstFlag] = 1 when some entry differs from
// its diagonal's sampled value (else every diagonal is one constant).
constexpr int kFarInfo = 10;
constexpr int kBandInfo = 16;
constexpr int kConstFlag = 13;
constexpr int kConstInfo = 32;   // int index; 8-byte aligned doubles
// further slots of the block, filled by other launches: the CSR check's two flags
// (launch_validate_csr) and the long rows' count (launch_long_rows)
constexpr int kCheckInfo = 56;
constexpr int kLongInfo = 58;
hipError_t launch_rows_probe(bool f64, const CsrDev& A, int* info, hipStream_t st);
hipError_t launch_dia_build(bool f64, const CsrDev& A, void* dia, uint16_t* pres, int* info, hipStream_t st);

// Alg. 2's stopping test after the step that produced w_m: for columns c < qc
// still active in *mask, e = |d_m| sqrt(sums[c*stride]) <= tol clears the bit
// and sets deg[c] = m (deg of the columns that never stop is left as set by
// the caller).  One wave; sums are FP64 column sums of w_m^2.
hipError_t launch_adapt_decide(const double* sums, int stride, int qc, double dm_abs, double tol, int m,
                               uint64_t* mask, int* deg, hipStream_t st);

// The column sums of a step's partials (nwg rows) and that test, in one launch.
hipError_t launch_reduce_decide(const double* part, int nwg, int qc, int part_ld, double dm_abs, double tol, int m,
                                uint64_t* mask, int* deg, hipStream_t st);

// The same test after `levels` steps taken together: level t = 0..levels-1
// produced w_{m+1+t}, sums[t*stride_t + c].  words (device): [0] the mask, in
// and out; [1 + t] the columns active before level t; [kAdaptNext + t] the new
// mask, for every t; [kAdaptRan] counts the calls that found an active column.
// *redo = 1 if some column stopped before the last level (it took terms that it
// should not have).  levels = 0 starts a loop: fills [kAdaptNext ..], clears
// [kAdaptRan]; sums[c * stride_t] is then the columns' own, and [kAdaptTop] their
// largest norm (as a double) over the active ones.
constexpr int kAdaptNext = 7, kAdaptTop = 14, kAdaptRan = 15, kAdaptWords = 16;
static_assert(kAdaptNext + kFusedMax <= kAdaptTop, "words of the levels");
struct AdaptLevels {
    double dm_abs[kFusedMax];
};
hipError_t launch_adapt_decide_levels(const double* sums, int stride_t, int qc, const AdaptLevels& lv, int levels,
                                      double tol, int m, uint64_t* words, int* redo, int* deg, hipStream_t st);

// Lanczos recurrence (lanczos.hip): step j of the FP64 recurrence on A, u = u_j,
// u_prev = u_{j-1}, w becomes u_{j+1} (all unnormalised); alpha[j], and beta of
// the step before, are written on the device.  launch_lanczos_beta writes
// beta[j] after step j.
constexpr int kLanczosWgs = 2048;
struct LanczosDev {
    int wgs;                      // lanczos_wgs(n): partial sums of part_a, part_b
    double *part_a, *part_b;
    double *alpha, *beta;
};
int lanczos_wgs(int n);
hipError_t launch_lanczos_start(int n, uint64_t key, double scale, double* u, hipStream_t st);
hipError_t launch_lanczos_step(bool f64, const CsrDev& A, const LanczosDev& d, const double* u, const double* u_prev,
                               double* w, int j, hipStream_t st);
hipError_t launch_lanczos_beta(const LanczosDev& d, int j, hipStream_t st);

}  // namespace ld
