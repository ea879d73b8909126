// Kernel argument blocks and launchers of libmsb (internal).
#pragma once

#include "common.h"

namespace msb {

enum { EPI_PLAIN = 0, EPI_MV = 1, EPI_MV_Y = 2, EPI_SV = 3, EPI_MVV = 4, EPI_MVN = 5, EPI_SV2 = 7 };
// epilogues that write partials (EPI_MVN: EPI_MV without the <r~, out> term,
// which a sparse list supplies; EPI_MVV: Re <v, out> in row 0 alone)
__host__ __device__ constexpr bool epi_dots(int e) { return e == EPI_MV || e == EPI_MVN || e == EPI_MVV; }

// A per-right-hand-side complex coefficient in device memory: the value for
// rhs r is *(const double2 *)(p + r * stride).
struct CoefRef {
    const char *p = nullptr;
    long stride = 0;
};
__device__ inline double2 ld(const CoefRef &c, int rhs) {
    return *(const double2 *)(c.p + (long)rhs * c.stride);
}

template <typename T>
struct DslashArgs {
    const C<T> *in = nullptr;
    C<T> *out = nullptr;
    const C<T> *U = nullptr;   // [4][3][3][V]
    Geom g{};
    T diag = 0, ef = 1, eb = 1, bc = -1;
    int g5out = 0;
    T scale = 1, sigma0 = 0;
    const double *sigma0_rhs = nullptr;  // if set: per-rhs sigma0 (overrides sigma0)
    const C<T> *v = nullptr;   // EPI_MV*: + sigma0 * v
    const C<T> *rt = nullptr;  // EPI_MV: partials of <rt, out>
    double *part = nullptr;    // [rhs][PMAX][ps]
    long ps = NBMAX;           // partial row stride
    int nsb = 0;               // site blocks (set by the launcher)
    int per = 0;               // blocks per XCD in the flattened grid (set by the launcher)
    int sstride = 0;           // site-loop stride (set by the launcher)
    int nrhs = 0;
    int nch = 0;               // chunked stencil: 64-site chunks (set by the launcher)
    int tsc = 0;               // chunked stencil: chunks per t-slice, 0 if not whole
    int per_t = 0;             // chunked stencil: blocks per XCD and group (per rounded up to tsc)
    int rpb = 0;               // chunked stencil: right-hand sides per block (set by the launcher)
    CoefRef ycoef;             // EPI_MV_Y: coefficient of the Mv output
    double2 *y = nullptr;      // EPI_MV_Y accumulator (always FP64)
    const C<T> *w = nullptr;   // EPI_SV2: subtracted from the output
    long w_rs = 0;
    Gate gate{};
    // element strides between right-hand sides (0: 12 V)
    long in_rs = 0, out_rs = 0, v_rs = 0, rt_rs = 0, y_rs = 0;
};

// The stencil on nrhs right-hand sides: picks the form (dslash_use_split) and
// sets its launch geometry.
template <typename T>
void launch_dslash(hipStream_t st, DslashArgs<T> a, int nrhs, int epi, bool g5in);
// Timing of the next launch_dslash on this host thread: its kernel is
// dispatched with start and stop events that the dispatch itself records
// (no event packets of their own on the stream around it).  stencil_timing_
// taken() reports, and clears, whether a launch consumed the pair.
void stencil_timing_arm(hipEvent_t start, hipEvent_t stop);
bool stencil_timing_taken();

// Geometry of the persistent kernel's stencil (256-site blocks): sets nsb,
// nrhs, per and sstride and returns the number of (virtual) blocks, 8 per, so that block p runs on
// XCD p % 8.
template <typename T>
inline long dslash_prepare(DslashArgs<T> &a, int nrhs) {
    a.nsb = (a.g.V + BLOCK - 1) / BLOCK;
    a.nrhs = nrhs;
    const long G = (long)a.nsb * nrhs;
    a.per = (int)((G + 7) / 8);
    a.sstride = 1 << 30;
    return 8L * a.per;
}

constexpr int CHUNK = 64;
constexpr int CHUNK_WAVES = 4;   // wavefronts per block of the chunked stencil
// Slabs of chunks per XCD (see slab_chunk).
template <typename T>
inline void dslash_slab_prepare(DslashArgs<T> &a, int nrhs) {
    a.nrhs = nrhs;
    a.nch = (a.g.V + CHUNK - 1) / CHUNK;
    a.per = (a.nch + 7) / 8;
    const int sites_t = a.g.Lx * a.g.Ly * a.g.Lz;
    a.tsc = (sites_t % CHUNK == 0) ? sites_t / CHUNK : 0;
    a.per_t = a.tsc ? ((a.per + a.tsc - 1) / a.tsc) * a.tsc : a.per;
}
// Which form: the split stencil (a block per chunk and right-hand side) for
// one right-hand side, which has no links to share, and below a number of
// blocks that depends on the epilogue; the chunked form beyond.  The more
// operands the epilogue reads beside the hops, the longer the split form's
// wider loads pay; with 2 or 3 right-hand sides the chunked form leaves
// wavefronts idle.  Launch times, split / chunked in us (FP64; FP32 has the
// same lines), on either side of each line:
//   at most v and w        2, 3 sources: 1944 blocks (12^3x24, EPI_SV) 24.8 / 27.0,
//                          2304 (16^3x12) 32.3 / 31.8, 3072 (16^3x24, plain) 41.1 / 34.6
//                          4 and more: 828 (10x9x7x14) 14.7 / 17.2, 1024 (8^3x32) 14.5 / 13.6
//   r~ (EPI_MV)            2, 3: 3072 (16^3x24) 44.6 / 46.5, 4096 (16^3x32) 68.2 / 61.9
//                          4 and more: 1944 (12^4) 31.8 / 36.4, 3072 (8^3x32) 41.5 / 39.0
//   y (EPI_MV_Y)           4096 (16^3x32, 2) 75.0 / 81.5, 3888 (12^4, 12) 60.5 / 77.2,
//                          4096 (16^4, 4) 63.2 / 61.0, 4608 (16^3x24, 3) 76.8 / 74.7
//   gamma5 on the input,   2, 3: 4608 (16^3x24) 47.0 / 52.3, 6144 (16^3x32) 78.8 / 71.0
//   FP64 (one wavefront    4 and more: 1024 (8^4) 14.2 / 11.6
//   per SIMD if chunked)
template <typename T, int EPI, bool G5IN>
constexpr bool dslash_use_split(long nch, int nrhs) {
    const bool few = nrhs < CHUNK_WAVES;
    long blocks = few ? 2048 : 1024;
    if (EPI == EPI_MV) blocks = few ? 3200 : 2048;
    if (EPI == EPI_MV_Y) blocks = 4200;
    if (G5IN && sizeof(T) == 8) blocks = few ? 4700 : 1024;
    return nrhs == 1 || nch * nrhs < blocks;
}
// Launch geometry of the split stencil; returns its number of blocks.
template <typename T>
inline long dslash_split_prepare(DslashArgs<T> &a, int nrhs) {
    dslash_slab_prepare(a, nrhs);
    return 8L * a.per_t * nrhs;
}
// Launch geometry of the chunked stencil; returns its number of blocks.
//
// One block per chunk sweeps every right-hand side while the chunks alone fill
// the chip (512 FP64 blocks at a time, by the 74 KB of links each stages and
// its registers).  Below 768 chunks each block takes at most one right-hand
// side per wavefront instead (balanced groups), staging its links again from
// the caches: EPI_MV, one group / groups, 12 sources on 8^4 (64 chunks) 30.0 /
// 15.7 us, on 12^3x24 (648) 103.9 / 98.3, 24 there 197.7 / 182.0; 12 on
// 16^3x12 (768) 119.2 / 120.4, on 16^4 (1024) 134.7 / 143.0.  With gamma5 on
// the input in FP64, one wavefront per SIMD, staging again costs more and the
// line lies at 256 chunks: 12 on 10x9x7x14 (138) 23.5 / 20.5, on 8^3x32 (256)
// 25.8 / 28.0, on 16^4 103.9 / 119.1.
template <typename T, bool G5IN>
inline long dslash_chunk_prepare(DslashArgs<T> &a, int nrhs) {
    dslash_slab_prepare(a, nrhs);
    a.sstride = 1 << 30;
    int groups = 1;
    if (a.nch < (G5IN && sizeof(T) == 8 ? 256 : 768)) groups = (nrhs + CHUNK_WAVES - 1) / CHUNK_WAVES;
    a.rpb = (nrhs + groups - 1) / groups;
    groups = (nrhs + a.rpb - 1) / a.rpb;
    return 8L * a.per_t * groups;
}

// link force: pairs (c, p, q), the gradient of sum c Re <p, D(mu) q>
struct LinkPair {
    const double2 *p = nullptr, *q = nullptr;
    long p_rs = 0, q_rs = 0;   // element strides between right-hand sides (0: 12 V)
    double c = 0;
    int g5p = 0;               // use gamma5 p instead of p
};
constexpr int MAX_PAIRS = 4;
struct LinkForceArgs {
    Geom g{};
    double ef = 1, eb = 1, bc = -1;
    int npair = 0, nrhs = 1;
    LinkPair pairs[MAX_PAIRS];
    double2 *G = nullptr;      // [4][3][3][V], accumulated (+=)
};
void launch_link_force(hipStream_t st, const LinkForceArgs &a);
// Per block of 256 links (U [4][3][3][V], 4V links), the largest Gershgorin
// bound max_k (Re M_kk + sum_{l != k} |M_kl|) of M = U^+ U over its links: an
// upper bound of ||U||_2^2 (exactly 1 up to rounding for unitary links).
// blockmax: device [nblk], nblk = ceil(4V / 256).
void launch_link_gershgorin(hipStream_t st, const double2 *U, int V, double *blockmax);
inline int link_gershgorin_blocks(int V) { return (4 * V + 255) / 256; }

// ---- vector kernels ------------------------------------------------------
template <typename T>
struct VecArgs {
    long n = 0;                 // elements (complex) per vector = 12 V
    int l = 0;                  // MR degree (vectors R_0..R_l, U_0..U_l)
    int nshift = 0;             // shifts per rhs in the shift arrays
    C<T> *R = nullptr;          // [rhs][l+1][n]
    C<T> *U = nullptr;          // [rhs][l+1][n]
    C<T> *W = nullptr;          // [rhs][nshift][l+1][n]  (pass 1)
    double2 *X = nullptr;       // [rhs][nshift][n] shift solutions, FP64 (pass 1)
    double2 *XH = nullptr;      // [rhs][n] seed solution, FP64 (reliable updates)
    const C<T> *rt = nullptr;   // [rhs][n] shadow residual
    double *part = nullptr;
    long ps = NBMAX;            // partial row stride
    const SeedState *seed = nullptr;
    const StepCoef *sc = nullptr;   // [rhs][NSMAX]
    const MRCoef *mc = nullptr;     // [rhs][NSMAX]
    CoefRef beta, alpha;
    CoefRef gam;                // gamma_1 at gam, gamma_i at gam.p + (i-1)*16
    int partials = 1;
    Gate gate{};
    // fused r-update whose own gate is closed: with this one open (its step
    // ended after its u-Mv) it makes the step's direction update alone
    Gate gate_u{};
    int has_gate_u = 0;
    // deferred single pass
    C<T> *Bm = nullptr;         // [rhs][2l+2][n] the outer iteration's basis
    C<T> *W0 = nullptr;         // [rhs][nshift][n] u^s_0 of every shift
    const DeferCoef *dc = nullptr;  // [rhs][NSMAX]
    // pseudo-double pass: an Mv output is written to the store only, and is
    // read from there (not from R / U) until its first update; index -1: none
    const C<T> *r_src = nullptr;
    long r_src_rs = 0;
    int r_src_i = -1;
    const C<T> *u_src = nullptr;
    long u_src_rs = 0;
    int u_src_i = -1;
    // the MR step of the pseudo-double pass and of the deferred single pass
    // (mr_dyn = 1): r_L and u_L, L the BiCG steps the outer iteration
    // completed, are read from the iteration's store slots (slot t at
    // st_base + rhs * st_rs + t n) unless a step updated them since: r_L
    // always (its first update would be step L's r-update), u_L unless step
    // L made its u-step before a gamma breakdown
    const C<T> *st_base = nullptr;
    long st_rs = 0;
    int mr_dyn = 0;
};

// Basis form of the seed (MSB_SEED_BASIS, FP64): the vectors of the basis
// kernels.  Vector b of the outer iteration's basis (see SeedBasis) of right-
// hand side r is at bv[b] + r * brs[b].
template <typename T>
struct BasisArgs {
    long n = 0;
    int l = 0;
    Gate gate{};
    const C<T> *bv[NBB] = {};
    long brs[NBB] = {};
    const SeedBasis *sb = nullptr;    // [rhs]
    const SeedState *seed = nullptr;
    double *part = nullptr;
    long ps = NBMAX;
    // axpy: dst = x - c y with c per right-hand side; ||dst||^2 into partial
    // row prow when prow >= 0
    C<T> *dst = nullptr;
    long dst_rs = 0;
    const C<T> *x = nullptr;
    long x_rs = 0;
    const C<T> *y = nullptr;
    long y_rs = 0;
    CoefRef c{};
    int prow = -1;
    // r_0 from the basis: the first nbu basis vectors, ||r_0||^2 into row 3
    int nbu = 0;
    // MR update: r_0 and u_0 written over B_0 and B_1; <r~, r_0> (rt, or left
    // at zero for the sparse list) and ||r_0||^2 into rows 0..2
    C<T> *R0 = nullptr;
    C<T> *U0 = nullptr;
    long r0_rs = 0, u0_rs = 0;
    const C<T> *rt = nullptr;
    // MR update with a sparse r~ (wu set): <r~, r_0> from r_0 at the list's
    // entries (into rows 0, 1), the next outer iteration's beta from it
    // (the state's beta_spec) and u_0 = r_0 - beta u_0 into wu ([rhs][n])
    C<T> *wu = nullptr;
    const long *sp_idx = nullptr;     // [rhs][sp_max]
    const double2 *sp_val = nullptr;  // [rhs][sp_max]
    const int *sp_cnt = nullptr;      // [rhs], at most SPARSE_MAX
    int sp_max = 0;
    // deferred single pass: the shifts' vectors, updated by the MR update
    C<T> *W0 = nullptr;               // [rhs][nshift][n] u^s_0 of every shift
    double2 *X = nullptr;             // [rhs][nshift][n] shift solutions
    const DeferCoef *dc = nullptr;    // [rhs][NSMAX]
    int nshift = 0;
};
void launch_basis_axpy(hipStream_t, const BasisArgs<double> &, int nrhs, int nblk);
// replay of the double pass in basis form: r_0, u_0 after outer iteration
// m from the basis with the coefficients of sc_basis_replay (sb[rhs].r[0],
// u[0], over the first sb[rhs].nbu basis vectors), written over B_0, B_1
void launch_basis_combine(hipStream_t, const BasisArgs<double> &, int nrhs, int nblk);
void launch_basis_r0norm(hipStream_t, const BasisArgs<double> &, int nrhs, int nblk);
void launch_basis_gram(hipStream_t, const BasisArgs<double> &, int nrhs, int nblk);
// shifts: also every active shift's update over the outer iteration
void launch_basis_mr_update(hipStream_t, const BasisArgs<double> &, bool shifts, int nrhs, int nblk);

// one: u_j only (see seed_u_body)
template <typename T> void launch_seed_u(hipStream_t, const VecArgs<T> &, int j, int nrhs, int nblk, bool one = false);
// fused: the r-update also applies the step's deferred u_0..u_{j-1} update
template <typename T>
void launch_r_update(hipStream_t, const VecArgs<T> &, int j, bool shifts, bool xh, int nrhs, int nblk,
                     bool fused = false);
template <typename T> void launch_gram(hipStream_t, const VecArgs<T> &, int nrhs, int nblk);
template <typename T> void launch_mr_update(hipStream_t, const VecArgs<T> &, bool shifts, bool xh, int nrhs, int nblk);
// reliable update: r_0 = b - v (v = S x in FP64), partials <rt, r_0>, ||r_0||^2
// (optionally y += c v with c from yc)
template <typename T> void launch_rel_update(hipStream_t, const VecArgs<T> &, const double2 *b, const double2 *v,
                                             double2 *y, CoefRef yc, int nrhs, int nblk);

// deferred single pass: B_0 <- r_0, B_1 <- u_0 at the start of an outer
// iteration; once per iteration, u^s_0 and x^s of every active shift from B
template <typename T> void launch_snapshot(hipStream_t, const VecArgs<T> &, int nrhs, int nblk);
template <typename T> void launch_defer_update(hipStream_t, const VecArgs<T> &, int nrhs, int nblk);

// pseudo-double pass: y += sum over outer iterations m0 .. m0+mc-1 of this
// storage chunk of cu V^u_{m,j} + cr V^r_{m,j} (replay coefficients, step flags)
// and, when rel is given, crel S x_m of the reliable updates.
// V: [rhs][chunk slots][2l][n] (v_rs between rhs); rel: [chunk slots][rhs][n]
// FP64 (rel_ms between slots).
template <typename T>
void launch_pstore_sum(hipStream_t, double2 *y, const C<T> *V, long v_rs, const double2 *rel, long rel_ms,
                       const ReplayStep *rs, const ReplayOuter *ro, int Mcap, int l, int m0, int mc, long n,
                       int nrhs, int nblk);

// small utility kernels
template <typename T>
void launch_convert_in(hipStream_t, C<T> *dst, const double2 *src, long n, long dst_stride,
                       long src_stride, int nrhs);
template <typename T>
void launch_convert_out(hipStream_t, double2 *dst, const C<T> *src, long n, long dst_stride,
                        long src_stride, int nrhs);
template <typename T>
void launch_zero(hipStream_t, C<T> *dst, long n, long stride, int nrhs);
void launch_zero_gated(hipStream_t, double2 *dst, long n, long stride, int nrhs, int nblk, Gate gate);

// sparse shadow residual: index list of the nonzero entries of v ([nrhs] rows
// of n at stride rs), at most spmax per row, in index order.  Returns the
// largest row count (the list is written only when it is <= spmax), or -1 on
// a HIP error.  work: nrhs * nb ints.  Synchronises the stream.
int sparse_list(hipStream_t, const double2 *v, long n, long rs, int nrhs, int spmax, long *idx, double2 *val,
                int *cnt, int *work, int nb, bool fp32 = false);
struct SparseVec {
    const long *idx = nullptr;      // [nrhs][spmax]
    const double2 *val = nullptr;   // [nrhs][spmax]
    const int *cnt = nullptr;       // [nrhs]
    int spmax = 0;
    const void *x = nullptr;        // the vector dotted with r~, rhs stride x_rs (elements); null: none
    long x_rs = 0;
    int fp32 = 0;                   // x holds float2 (mixed precision)
};
struct SparseDotArgs : SparseVec {
    const double2 *b = nullptr;     // set: dot with b - v instead (FP64, rhs stride x_rs)
    const double2 *v = nullptr;
    double *part = nullptr;
    long ps = 0;
    Gate gate{};
};
void launch_sparse_dot(hipStream_t, const SparseDotArgs &, int nrhs);
template <typename T>
void launch_dot_partials(hipStream_t, const C<T> *x, const C<T> *y, long n, double *part, long ps,
                         int nrhs, int nblk, Gate gate);
template <typename T>
void launch_diffnorm_partials(hipStream_t, const C<T> *x, const C<T> *y, long n, long sx, long sy,
                              double *part, long ps, int nrhs, int nblk);
// y[rhs] = sum_s w[rhs][s] X[rhs][s]   (X stride n per shift, nshift per rhs)
void launch_ysum(hipStream_t, double2 *y, const double2 *X, const double *w, long n, int nshift,
                 int nrhs, int nblk);
// per (rhs, shift): Re <eta_r, x_rs> and Re <z_rs, x_rs> partials into
// out[((rhs * ns + s) * 2 + k) * nblk + block]
void launch_shift_dots(hipStream_t, const double2 *eta, const double2 *X, const double2 *Z, long n, int ns,
                       int nrhs, int nblk, double *out);
// R[rhs] = b[rhs] - t[rhs] (b rows b_rs apart, t and R rows n apart),
// partial slot 0 = ||R||^2
void launch_residual(hipStream_t, double2 *R, const double2 *b, long b_rs, const double2 *t, long n,
                     double *part, long ps, int nrhs, int nblk);
// y[rhs] = c[rhs] * b[rhs]
void launch_yinit(hipStream_t, double2 *y, const double2 *b, const double2 *c, long n, int nrhs,
                  int nblk);
// out = b + gamma5 w   (overlap), or out = s * w
void launch_overlap_out(hipStream_t, double2 *out, const double2 *b, const double2 *w, long V,
                        int nrhs, int overlap, double s, int nblk);
// vector axpy with a host scalar: y += a * x over n complex
void launch_axpy_host(hipStream_t, double2 *y, const double2 *x, double2 a, long n, int nblk);

// ---- scalar (single block per rhs) kernels --------------------------------
struct ScalarArgs {
    SeedState *seed = nullptr;
    ShiftState *sh = nullptr;       // [rhs][NSMAX]
    StepCoef *sc = nullptr;
    MRCoef *mc = nullptr;
    TapeStep *tape = nullptr;       // [rhs][max_steps]
    double2 *tape_gam = nullptr;    // [rhs][max_outer][LMAX]
    TapeOuter *tape_outer = nullptr;  // [rhs][max_outer]
    const double *part = nullptr;
    long ps = NBMAX;                // partial row stride
    int nblk = 0;                   // blocks that wrote the partials consumed
    int nblk2 = 0;                  // blocks of the second partial source
    int l = 0;
    int j = 0;
    int record = 0;                 // record the tape (double-pass)
    StepCoef *sc_hist = nullptr;    // deferred: [rhs][LMAX][NSMAX] every step's shift coefficients
    DeferCoef *dc = nullptr;        // deferred: [rhs][NSMAX] the iteration's coefficients
    int shadow = 0;                 // init: ||r~|| from partial row 5 (r~ other than b)
    // basis form (MSB_SEED_BASIS)
    int basis = 0;
    int spec = 0;                   // the MR update forms the next u_0 update (sparse r~)
    double norm_a = 0;              // an upper bound of ||S|| (2-norm)
    SeedBasis *sb = nullptr;        // [rhs]
    // one-launch stages: the work of the next scalar stage on the same launch
    SparseVec sp;                   // sc_beta (j >= 1), sc_alpha: <r~, x> from r~'s list (x set)
    int then_beta = 0;              // sc_conv: then the next outer iteration's sc_beta (j = 0)
    int then_basis = 0;             // sc_alpha: then sc_basis (the last step of the outer iteration)
    int then_defer = 0;             // sc_mr: then sc_defer
};

void launch_sc_init(hipStream_t, const ScalarArgs &, int nrhs);
void launch_sc_beta(hipStream_t, const ScalarArgs &, int nrhs);
void launch_sc_alpha(hipStream_t, const ScalarArgs &, int nrhs);
// spec: then basis_spec (sparse r~, basis form)
void launch_sc_mr(hipStream_t, const ScalarArgs &, const BasisArgs<double> *spec, int nrhs);
void launch_sc_conv(hipStream_t, const ScalarArgs &, int nrhs);
void launch_sc_rel(hipStream_t, const ScalarArgs &, int nrhs);
// Replay of the double pass in basis form: outer iteration m's recorded step
// coefficients and MR coefficients (rs [rhs][Mcap][l], ro [rhs][Mcap]) as the
// combined coefficients of r_0 and u_0 after the iteration (sb[rhs])
struct BasisReplayArgs {
    const ReplayStep *rs = nullptr;
    const ReplayOuter *ro = nullptr;
    int Mcap = 0, l = 0, m = 0;
    SeedBasis *sb = nullptr;
};
void launch_sc_basis_replay(hipStream_t, const BasisReplayArgs &, int nrhs);
void launch_sc_exh(hipStream_t, const ScalarArgs &, int nrhs);

// ---- persistent execution --------------------------------------------------
// The stages of a solve, recorded as a table of operations that one
// cooperative launch executes in order, with a grid-wide barrier between
// consecutive operations.  Each operation is split into virtual blocks (the
// blocks its own launch would have had); resident block b takes the virtual
// blocks b, b + P, b + 2P, ... (P, the resident grid, is a multiple of 8, so
// a virtual block stays on the XCD its own launch would have used).
enum OpKind : int {
    OP_DS = 1,        // stencil in the iteration's precision (blob: DslashArgs<T>)
    OP_DS64,          // FP64 stencil of a reliable update (blob: DslashArgs<double>)
    OP_SEED_U,        // blob: VecArgs<T>
    OP_R_UPDATE,
    OP_GRAM,
    OP_MR_UPDATE,
    OP_REL_UPDATE,
    OP_SC_BETA,       // blob: ScalarArgs
    OP_SC_ALPHA,
    OP_SC_MR,
    OP_SC_REL,
    OP_SC_CONV,
    OP_SC_EXH,        // per-stage launches only (the basis form of the seed)
};
constexpr int POP_BLOB = 512;
struct alignas(16) POp {
    int kind = 0;
    int cls = 0;                 // timing class
    int epi = 0;                 // OP_DS, OP_DS64
    int j = 0;                   // OP_SEED_U, OP_R_UPDATE: BiCG step
    int shifts = 0;              // OP_R_UPDATE, OP_MR_UPDATE: update the shift vectors
    int nvb = 0;                 // virtual blocks
    int nblk = 0;                // vector ops: element blocks per right-hand side
    int pad = 0;
    const double2 *b = nullptr;  // OP_REL_UPDATE operands
    const double2 *v = nullptr;
    double2 *y = nullptr;
    CoefRef yc{};
    alignas(16) unsigned char blob[POP_BLOB];
};
constexpr int PERSIST_CLASSES = 8;
constexpr int PERSIST_GROUP = 32;      // blocks per first-level barrier group
constexpr int PERSIST_MAX_GROUPS = 64; // per XCD
// Barrier and timing state of a persistent launch (zeroed before it).
struct PersistCtl {
    unsigned long long bar;                              // XCD arrivals (one per XCD in use)
    int abort;                                           // set when a wait exceeds its bound
    int pad;
    unsigned long long ticks[PERSIST_CLASSES];           // wall-clock ticks per timing class
    unsigned long long execs[PERSIST_CLASSES];           // operations executed per class
    unsigned long long xbar[8], xrel[8];                 // per XCD: group arrivals, release
    unsigned long long gbar[8 * PERSIST_MAX_GROUPS];     // per group: block arrivals
    unsigned long long grel[8 * PERSIST_MAX_GROUPS];     // per group: release
    unsigned long long xcount[8];                        // census: blocks found on each XCD
    unsigned long long census;                           // census: blocks counted
};
struct PersistArgs {
    const POp *ops = nullptr;
    int nops = 0;                // operations per iteration of the table
    int iters = 1;               // repetitions of the table
    int loop = 0;                // 1: stop after a repetition when no seed runs
    const SeedState *seed = nullptr;
    int nrhs = 0;
    int timing = 0;              // record per-class stage times
    PersistCtl *ctl = nullptr;
};
// Largest co-resident grid of the persistent kernel of MR degree l (a
// multiple of 8; 0 when l is outside 1..PERSIST_LMAX).
constexpr int PERSIST_LMAX = 6;
template <typename T> int persistent_grid(int device, int l);
template <typename T> hipError_t launch_persistent(hipStream_t st, const PersistArgs &pa, int grid, int l);

}  // namespace msb
