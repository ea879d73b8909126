// Device bodies of the scalar stages of multi-shift BiCGstab(l), one block
// per right-hand side (see scalar.hip for the recurrences).  Shared by the
// one-launch-per-stage kernels (NT = SC_THREADS work-items) and the persistent
// kernel (NT = BLOCK).
#pragma once
#include "blas_dev.h"
#include "common.h"
#include "kernels.h"

namespace msb {
namespace dev {

__device__ inline const double *prow(const ScalarArgs &a, int rhs) {
    return a.part + (size_t)rhs * PMAX * a.ps;
}

// Work-items of the one-launch scalar stages.  These kernels are a few
// dependent trips to memory in one block per right-hand side; sixteen
// wavefronts take the rows of partial sums side by side.
constexpr int SC_THREADS = 1024;

// The state of one right-hand side as a scalar stage works on it.  The
// one-launch stages (NT > BLOCK) hold it in LDS: every word is loaded by a
// work-item of its own at the start, beside the partials and before any gate
// is known, and stored back at the end (leave), unchanged where the stage's
// gate was closed.
// Read field by field, each dependent read (gate, list of active shifts,
// shift) was a trip to memory of its own, since another XCD wrote it (with the
// MR stage's factor in registers: 8^4 at l = 4, MR 15.5 us, now 13.5, alpha
// 5.1, now 4.8; the overlap on 12^3x24 33.1 ms, now 32.3).
// The persistent kernel (NT == BLOCK) works on the state in place.
struct StateLds {
    SeedState s;
    ShiftState h[NSMAX];
};
template <int NT>
struct StageState {
    typedef unsigned long long __attribute__((may_alias)) Word;
    static constexpr int WS = sizeof(SeedState) / 8, W = sizeof(StateLds) / 8, PER = (W + NT - 1) / NT;
    static_assert(sizeof(SeedState) % 16 == 0 && sizeof(StateLds) == sizeof(SeedState) + NSMAX * sizeof(ShiftState),
                  "the two arrays' words follow each other");
    SeedState &S;
    ShiftState *H;
    Word *seed, *shifts;   // in memory
    Word v[PER];
    __device__ __forceinline__ StageState(const ScalarArgs &a, int rhs, StateLds &l)
        : S(l.s), H(l.h), seed(reinterpret_cast<Word *>(a.seed + rhs)),
          shifts(reinterpret_cast<Word *>(a.sh + (size_t)rhs * NSMAX)) {
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int w = threadIdx.x + p * NT;
            if (w < W) v[p] = w < WS ? seed[w] : shifts[w - WS];
        }
    }
    // the state is in LDS for every work-item
    __device__ __forceinline__ void arrive() {
        Word *d = reinterpret_cast<Word *>(&S);
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int w = threadIdx.x + p * NT;
            if (w < W) d[w] = v[p];
        }
        __syncthreads();
    }
    // arrive, and whether BiCG steps go on: read by every wavefront before any
    // may write it (a stage that breaks down clears bicg_on, and a wavefront
    // that found it cleared would leave the others at their next barrier)
    __device__ __forceinline__ bool arrive_bicg() {
        arrive();
        const bool on = S.run && S.bicg_on;
        __syncthreads();
        return on;
    }
    // after the last write to it (every work-item calls it)
    __device__ __forceinline__ void leave() {
        __syncthreads();
        const Word *d = reinterpret_cast<const Word *>(&S);
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            const int w = threadIdx.x + p * NT;
            if (w < W) (w < WS ? seed[w] : shifts[w - WS]) = d[w];
        }
    }
};
template <>
struct StageState<BLOCK> {
    SeedState &S;
    ShiftState *H;
    __device__ __forceinline__ StageState(const ScalarArgs &a, int rhs)
        : S(a.seed[rhs]), H(a.sh + (size_t)rhs * NSMAX) {}
    __device__ __forceinline__ void arrive() {}
    __device__ __forceinline__ bool arrive_bicg() { return true; }   // tested before the sums, whose barriers follow
};

// sums of rows rows[0 .. cnt) of the partials, as block_sum gives each
template <int NT, int NR>
__device__ inline void sum_rows(const double *row, long ps, const int *rows, int cnt, int n, double (&out)[NR]) {
    if constexpr (NT == BLOCK) block_sum_rows<NR>(row, ps, rows, cnt, n, out);
    else block_sum_rows_wide<NT, NR>(row, ps, rows, cnt, n, out);
}
// the sum of one row
template <int NT>
__device__ inline double sum1(const double *row, int n) {
    if constexpr (NT == BLOCK) {
        return block_sum(row, n);
    } else {
        const int rows[1] = {0};
        double o[1];
        block_sum_rows_wide<NT, 1>(row, 0, rows, 1, n, o);
        return o[0];
    }
}
// the sums of partial rows 0, 1, 2 (re, im of an inner product, a squared norm)
template <int NT>
__device__ inline void sum3(const double *row, long ps, int n, double &s0, double &s1, double &s2) {
    const int rows[3] = {0, 1, 2};
    double o[3];
    sum_rows<NT, 3>(row, ps, rows, 3, n, o);
    s0 = o[0];
    s1 = o[1];
    s2 = o[2];
}

// min over the active shifts of |zeta psi| (1e308 without any), for wavefront
// 0: a shift per lane (NSMAX = 64 of them), since one lane's walk over the
// shifts' states was a chain of trips to memory
__device__ inline double min_shift_scale(const SeedState &S, const ShiftState *Hs) {
    static_assert(NSMAX == 64, "one shift per lane");
    double mn = 1e308;
    const int q = threadIdx.x & 63;
    if (q < S.nact) {
        const ShiftState &H = Hs[S.act[q]];
        if (H.active) {
            const double sc = cmod(cmul(H.zeta, H.psi));
            mn = sc < mn ? sc : mn;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(mn, off, 64);
        mn = o < mn ? o : mn;
    }
    return mn;
}

__device__ __forceinline__ void sc_init_body(const ScalarArgs &a, int rhs) {
    SeedState &S = a.seed[rhs];
    const double *row = prow(a, rhs);
    const double re = block_sum(row, a.nblk);
    const double im = block_sum(row + a.ps, a.nblk);
    const double nb2 = block_sum(row + 2 * a.ps, a.nblk);
    const double rt2 = a.shadow ? block_sum(row + 5 * a.ps, a.nblk) : nb2;
    if (threadIdx.x == 0) {
        S.rho1 = d2(re, im);
        S.bnorm = sqrt(nb2);
        S.rtnorm = sqrt(rt2);
        S.rnorm0 = S.bnorm;
        S.rnorm_j = S.bnorm;
        S.rho0 = d2(1, 0);
        S.alpha = d2(0, 0);
        S.omega = d2(1, 0);
        S.beta = d2(0, 0);
        for (int i = 0; i < LMAX; ++i) S.gam[i] = d2(0, 0);
        S.bicg_on = 1;
        S.l_eff = 0;
        S.l_mr = 0;
        S.broken = S.exhausted = S.partial = 0;
        S.m = S.n = 0;
        S.status = S_OK;
        S.mv = S.dots = S.axpys = S.reliable = 0;
        S.rel = 0;
        S.rmax = S.bnorm;
        S.beta_spec = d2(NAN, NAN);
        S.wu_ready = 0;
        for (int i = 0; i < LMAX; ++i) S.step_flag[i] = 0;
        S.nact = 0;
        for (int s = 0; s < S.nshift; ++s) {
            if (a.sh[(size_t)rhs * NSMAX + s].active) S.act[S.nact++] = s;
        }
        S.dots = 0;
        S.run = (S.bnorm > 0.0 && S.nact > 0 && isfinite(S.bnorm)) ? 1 : 0;
        if (!isfinite(S.bnorm)) S.status = S_ERR_ARG;
        if (!(S.bnorm > 0.0) || !isfinite(S.bnorm)) {
            for (int s = 0; s < S.nshift; ++s) {
                ShiftState &H = a.sh[(size_t)rhs * NSMAX + s];
                H.active = 0;
                H.iters = 0;
                H.res = 0.0;
            }
            S.nact = 0;
        }
    }
}

// <r~, x> from the list of r~'s nonzero entries, each product formed in FP64
// as the dense epilogues do.  A lane of wavefront 0 per entry loads it and x
// there (its entry before the count is known), then every work-item adds the
// products in the list's order.
template <typename X>
__device__ inline double2 sparse_sum(const SparseVec &v, int rhs) {
    __shared__ double2 ts[SPARSE_MAX], zs[SPARSE_MAX];
    const int nk = v.cnt[rhs], k0 = threadIdx.x;
    if (k0 < v.spmax && k0 < SPARSE_MAX) {
        const double2 t = v.val[(size_t)rhs * v.spmax + k0];
        const auto e = v.idx[(size_t)rhs * v.spmax + k0];
        if (k0 < nk) {
            const X z = reinterpret_cast<const X *>(v.x)[(size_t)rhs * v.x_rs + e];
            ts[k0] = t;
            zs[k0] = d2((double)z.x, (double)z.y);
        }
    }
    __syncthreads();
    double p0 = 0.0, p1 = 0.0;
    for (int k = 0; k < nk; ++k) {
        const double2 t = ts[k], z = zs[k];
        p0 += t.x * z.x + t.y * z.y;
        p1 += t.x * z.y - t.y * z.x;
    }
    return d2(p0, p1);
}
// sum3, with <r~, x> from the list where the stage has one (the rows 0 and 1
// are zero then): a launch of its own for that took 4.7 us after every Mv
template <int NT>
__device__ inline void dot_sums(const ScalarArgs &a, int rhs, double &re, double &im, double &n2) {
    const double *row = prow(a, rhs);
    if (NT != BLOCK && a.sp.x) {
        const double2 d = a.sp.fp32 ? sparse_sum<float2>(a.sp, rhs) : sparse_sum<double2>(a.sp, rhs);
        re = d.x;
        im = d.y;
        n2 = sum1<NT>(row + 2 * a.ps, a.nblk);
    } else {
        sum3<NT>(row, a.ps, a.nblk, re, im, n2);
    }
}

// beta of BiCG step j from rho_1 = <r~, r_j> and ||r_j||^2 (one work-item)
__device__ __forceinline__ void beta_step(const ScalarArgs &a, SeedState &S, int rhs, int j, double2 rho1,
                                          double rj2) {
    if (j == 0) {
        S.wu_ready = 0;
        S.rho0 = cneg(cmul(S.omega, S.rho0));
    }
    S.dots += 1;
    if ((rho1.x == 0.0 && rho1.y == 0.0) || !cfinite(rho1) ||
        cabsd(rho1) <= BREAK_REL * S.rtnorm * sqrt(rj2)) {
        S.broken = 1;
        S.bicg_on = 0;
        S.l_eff = j;
        return;
    }
    const double2 beta = cdiv(cmul(S.alpha, rho1), S.rho0);
    if (j == 0 && a.spec) {
        // the MR update already made u_0 = r_0 - beta u_0 with this beta
        S.wu_ready = (beta.x == S.beta_spec.x && beta.y == S.beta_spec.y) ? 1 : 0;
        S.beta_spec = d2(NAN, NAN);
    }
    S.rho0 = rho1;
    S.beta = beta;
    S.step_beta[j] = beta;
    S.step_flag[j] = 1;
    if (a.record && S.n < S.max_steps) {
        TapeStep &t = a.tape[(size_t)rhs * S.max_steps + S.n];
        t.beta = beta;
        t.alpha = d2(0, 0);
        t.flag = 0;
    }
}

template <int NT>
__device__ __forceinline__ void sc_beta_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    if (NT == BLOCK && (!S.run || !S.bicg_on)) return;
    const int j = a.j;
    const double *row = prow(a, rhs);
    double re, im, rj2, r02 = 0.0;
    dot_sums<NT>(a, rhs, re, im, rj2);
    // basis form: ||r_0|| exists only where sc_exh found that the test could
    // fire; elsewhere it cannot (||r_0|| >= ||r_{j-1}|| / ||S||^(j-1))
    if (NT != BLOCK) {
        if (j >= 1 && !a.basis) r02 = sum1<NT>(row + 3 * a.ps, a.nblk2);
        if (!st.arrive_bicg()) return;
    }
    const bool have_r0 = !a.basis || S.exh_check;
    const bool test = j >= 1 && have_r0 && !S.forced && S.nact > 0;
    if (j >= 1 && have_r0 && (NT == BLOCK || a.basis)) r02 = sum1<NT>(row + 3 * a.ps, a.nblk2);
    if (threadIdx.x >= 64) return;
    const double mn = test ? min_shift_scale(S, st.H) : 0.0;
    if (threadIdx.x != 0) return;
    if (j >= 1 && have_r0) S.rnorm0 = sqrt(r02);
    if (test) {
        // Krylov space exhausted: every active shift already meets its
        // tolerance after the previous step's r-update
        if (S.rnorm0 <= FREEZE_FRAC * S.tol * S.bnorm * mn) {
            S.exhausted = 1;
            S.bicg_on = 0;
            S.l_eff = j;
            return;
        }
    }
    beta_step(a, S, rhs, j, d2(re, im), rj2);
}

template <int NT>
__device__ __forceinline__ void sc_alpha_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    if (NT == BLOCK && (!S.run || !S.bicg_on)) return;
    const int j = a.j;
    double re, im, u2;
    dot_sums<NT>(a, rhs, re, im, u2);
    if (!st.arrive_bicg()) return;
    __shared__ int ok;
    __shared__ double2 sh_alpha, sh_beta;
    if (threadIdx.x == 0) {
        const double2 gam = d2(re, im);
        S.dots += 1;
        S.mv += 1;
        ok = 1;
        if ((gam.x == 0.0 && gam.y == 0.0) || !cfinite(gam) ||
            cabsd(gam) <= BREAK_REL * S.rtnorm * sqrt(u2)) {
            S.broken = 1;
            S.partial = 1;
            S.bicg_on = 0;
            S.l_eff = j;
            if (a.record && S.n < S.max_steps) a.tape[(size_t)rhs * S.max_steps + S.n].flag = 1;
            ok = 0;
        } else {
            const double2 alpha = cdiv(S.rho0, gam);
            S.alpha = alpha;
            S.step_alpha[j] = alpha;
            S.step_flag[j] = 2;
            if (a.record && S.n < S.max_steps) {
                TapeStep &t = a.tape[(size_t)rhs * S.max_steps + S.n];
                t.alpha = alpha;
                t.flag = 2;
            }
        }
        sh_alpha = S.alpha;
        sh_beta = S.beta;
    }
    __syncthreads();
    if (!ok) return;
    const double2 alpha = sh_alpha, beta = sh_beta;
    const int nact = S.nact;
    for (int q = threadIdx.x; q < nact; q += BLOCK) {
        const int s = S.act[q];
        ShiftState &H = st.H[s];
        StepCoef &c = a.sc[(size_t)rhs * NSMAX + q];
        c.s = s;
        if (!H.active) {
            c.live = 0;
            continue;
        }
        const double2 z = H.zeta, zp = H.zeta_prev, pp = H.pi_prev, ps = H.psi;
        const double sp = H.sp;
        const double2 pi_n = csub(z, cmul(beta, pp));
        const double2 step = cscale(cmul(alpha, pi_n), sp);
        const double2 z_next = cadd(z, step);
        // zeta_{n+1} not finite or cancelled to rounding: the shifted
        // recurrence has no next iterate (broken); |zeta_{n+1} psi| beyond
        // ZETA_MAX: converged
        const bool brk = !cfinite(z_next) || cmod(z_next) < ZETA_MIN ||
                         cmod(z_next) <= BREAK_REL * (cmod(z) + cmod(step));
        if (brk || !(cmod(z_next) * cmod(ps) <= ZETA_MAX)) {
            H.active = 0;
            H.broken = brk ? 1 : 0;
            H.stopped = 1;
            H.iters = S.m;
            c.live = 0;
            continue;
        }
        const double2 alpha_s = cdiv(cmul(alpha, z), z_next);
        const double2 rz = cdiv(zp, z);
        const double2 beta_s = cmul(beta, cmul(rz, rz));
        const double2 kap = cdiv(d2(1, 0), cmul(z, ps));
        const double2 kap_next = cdiv(d2(1, 0), cmul(z_next, ps));
        c.kap = kap;
        c.beta_s = beta_s;
        c.alpha_s = alpha_s;
        c.a1 = cdiv(csub(kap, kap_next), alpha_s);
        c.a2 = cdiv(cmul(kap_next, alpha), alpha_s);
        c.sp = sp;
        c.live = 1;
        H.zeta_prev = z;
        H.zeta = z_next;
        H.pi_prev = pi_n;
    }
    if (a.sc_hist) {
        // deferred single pass: keep every step's coefficients of the iteration
        __syncthreads();
        for (int q = threadIdx.x; q < nact; q += BLOCK)
            a.sc_hist[((size_t)rhs * LMAX + j) * NSMAX + q] = a.sc[(size_t)rhs * NSMAX + q];
    }
    if (threadIdx.x == 0) {
        S.mv += 1;
        S.n += 1;
        S.l_eff = j + 1;
    }
}

// The factorisation has two forms, registers and LDS, that have to give the
// same bits.  rounded: x, which the compiler may not fuse with what it goes
// into (a product into a difference, a root into a reciprocal root).  Then
// acc - a conj(b), acc - a b and acc - conj(a) b with the product fused as the
// compiler does in the LDS form, whose loops leave it no other choice.
__device__ inline double rounded(double x) {
    asm("" : "+v"(x));
    return x;
}
__device__ inline double2 rounded(double2 x) { return d2(rounded(x.x), rounded(x.y)); }
__device__ inline double2 sub_mulc(double2 acc, double2 a, double2 b) {
    return d2(acc.x - __builtin_fma(a.x, b.x, a.y * b.y), acc.y - __builtin_fma(a.y, b.x, -(a.x * b.y)));
}
__device__ inline double2 sub_mul(double2 acc, double2 a, double2 b) {
    return d2(acc.x - __builtin_fma(a.x, b.x, -(a.y * b.y)), acc.y - __builtin_fma(a.y, b.x, a.x * b.y));
}
__device__ inline double2 sub_cmul(double2 acc, double2 a, double2 b) {
    return d2(acc.x - __builtin_fma(a.x, b.x, a.y * b.y), acc.y - __builtin_fma(a.x, b.y, -(a.y * b.x)));
}

// LT: the compile-time l of a one-launch stage, 0 in the persistent kernel
template <int LT, int NT>
__device__ __forceinline__ void sc_mr_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    if (NT == BLOCK && !S.run) return;
    const int l = a.l;
    // terms to sum: those of the steps taken, or all l where the sums are
    // formed before the state has arrived (the others are not used)
    int L = l;
    if (NT == BLOCK) L = S.exhausted ? 0 : S.l_eff;
    __shared__ double2 G[LMAX][LMAX];
    __shared__ double2 cvec[LMAX];
    __shared__ double2 g[LMAX];
    // the Cholesky factor and the forward-substitution vector, used by
    // thread 0 alone: in LDS, since indexed at run time they would otherwise
    // live in scratch memory, whose dependent accesses dominated the kernel
    __shared__ double2 Lm[LMAX][LMAX];
    __shared__ double2 zz[LMAX];
    __shared__ int lmr_sh;
    const double *row = prow(a, rhs);
    // pair index of (i, k), i <= k, in the gram kernel's order over 0..l
    auto pidx = [l](int i, int k) {
        int p = 0;
        for (int ii = 0; ii < i; ++ii) p += l + 1 - ii;
        return p + (k - i);
    };
    if constexpr (NT == BLOCK) {
        // the pairs (i, k) in the Gram kernel's order, 4 pairs (8 partial rows)
        // per pass over the partials (more would cost the persistent kernel, which
        // inlines this body, an occupancy step)
        constexpr int NB = 4;
        int pi_[NB], pk_[NB], rows[2 * NB];
        int cnt = 0;
        for (int i = 0; i <= L; ++i) {
            for (int k = (i == 0 ? 1 : i); k <= L; ++k) {
                pi_[cnt] = i;
                pk_[cnt] = k;
                rows[2 * cnt] = 2 * pidx(i, k);
                rows[2 * cnt + 1] = 2 * pidx(i, k) + 1;
                ++cnt;
                const bool last = i == L && k == L;
                if (cnt == NB || last) {
                    double sums[2 * NB];
                    block_sum_rows<2 * NB>(row, a.ps, rows, 2 * cnt, a.nblk, sums);
                    if (threadIdx.x == 0) {
                        for (int q = 0; q < cnt; ++q) {
                            const double re = sums[2 * q], im = sums[2 * q + 1];
                            if (pi_[q] == 0) {
                                cvec[pk_[q] - 1] = d2(re, -im);   // <r_k, r_0> = conj(<r_0, r_k>)
                            } else {
                                G[pi_[q] - 1][pk_[q] - 1] = d2(re, im);
                                G[pk_[q] - 1][pi_[q] - 1] = d2(re, -im);
                            }
                        }
                    }
                    cnt = 0;
                }
            }
        }
    } else {
        // every pair at once: a wavefront per piece of a row (at most 44
        // pairs), the loads of TB pieces in flight together (one piece at a
        // time was a chain of trips to memory: 35 us at l = 6 on 24^3x48, now
        // 28, the rest the serial factorisation)
        constexpr int NPX = (LMAX + 1) * (LMAX + 2) / 2, NW = NT / 64, TB = 4, UP = 8;
        static_assert(NW % 4 == 0, "a wavefront's pieces are the same quarter of their rows");
        __shared__ double sh[2 * NPX][4];
        const int lane = threadIdx.x & 63, np = (L + 1) * (L + 2) / 2;
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        // pieces 0 .. 7 are ||r_0||^2, which is not part of the system
        for (int t0 = 8 + wave; t0 < 8 * np; t0 += TB * NW) {
            const double *pr[TB];
            double x[TB];
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                // pair number -> (i, k) over 0..L, its row in the kernel's numbering over 0..l
                const int task = t0 + b * NW < 8 * np ? t0 + b * NW : t0;
                int i = 0, q = task >> 3;
                while (q > L - i) {
                    q -= L + 1 - i;
                    ++i;
                }
                pr[b] = row + (size_t)(2 * pidx(i, i + q) + ((task >> 2) & 1)) * a.ps;
                x[b] = 0.0;
            }
            for (int e = (t0 & 3) * 64 + lane; e < a.nblk; e += UP * BLOCK) {
                double v[TB][UP];
#pragma unroll
                for (int b = 0; b < TB; ++b)
#pragma unroll
                    for (int u = 0; u < UP; ++u) v[b][u] = e + u * BLOCK < a.nblk ? pr[b][e + u * BLOCK] : 0.0;
#pragma unroll
                for (int b = 0; b < TB; ++b)
#pragma unroll
                    for (int u = 0; u < UP; ++u) x[b] += v[b][u];
            }
            const double s = wave_sums<TB>(x);
            const int b = wave_sums_index(), task = t0 + b * NW;
            if (b < TB && task < 8 * np) sh[task >> 2][task & 3] = s;
        }
        st.arrive();
        if (!S.run) return;
        if ((int)threadIdx.x < np) {
            int i = 0, q = threadIdx.x;
            while (q > L - i) {
                q -= L + 1 - i;
                ++i;
            }
            const int k = i + q;
            if (k > 0) {
                const double *s0 = sh[2 * threadIdx.x], *s1 = sh[2 * threadIdx.x + 1];
                const double re = ((s0[0] + s0[1]) + s0[2]) + s0[3], im = ((s1[0] + s1[1]) + s1[2]) + s1[3];
                if (i == 0) {
                    cvec[k - 1] = d2(re, -im);   // <r_k, r_0> = conj(<r_0, r_k>)
                } else {
                    G[i - 1][k - 1] = d2(re, im);
                    G[k - 1][i - 1] = d2(re, -im);
                }
            }
        }
        L = S.exhausted ? 0 : S.l_eff;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int n = L;
        int kok = n;
        if constexpr (LT > 0) {
            // the factor in registers, every loop unrolled: through LDS each
            // operand was a dependent trip (rows from n on are formed where
            // that needs no branch, and not used)
            double dmax = 0.0;
            for (int i = 0; i < n; ++i) dmax = G[i][i].x > dmax ? G[i][i].x : dmax;
            double2 F[LT][LT], z[LT], x[LT];
            double inv[LT];
#pragma unroll
            for (int i = 0; i < LT; ++i) {
                if (i >= kok) continue;
                double d = G[i][i].x;
#pragma unroll
                for (int p = 0; p < i; ++p) d -= __builtin_fma(F[i][p].x, F[i][p].x, F[i][p].y * F[i][p].y);
                if (!(d > CHOL_REL * dmax)) {
                    kok = i;
                    continue;
                }
                inv[i] = 1.0 / rounded(sqrt(d));
#pragma unroll
                for (int r = i + 1; r < LT; ++r) {
                    double2 acc = G[r][i];
#pragma unroll
                    for (int p = 0; p < i; ++p) acc = sub_mulc(acc, F[r][p], F[i][p]);
                    F[r][i] = rounded(cscale(acc, inv[i]));
                }
            }
            n = kok;
#pragma unroll
            for (int i = 0; i < LT; ++i) {
                if (i >= n) continue;
                double2 acc = cvec[i];
#pragma unroll
                for (int p = 0; p < i; ++p) acc = sub_mul(acc, F[i][p], z[p]);
                z[i] = rounded(cscale(acc, inv[i]));
            }
#pragma unroll
            for (int i = LT - 1; i >= 0; --i) {
                if (i >= n) continue;
                double2 acc = z[i];
#pragma unroll
                for (int p = i + 1; p < LT; ++p)
                    if (p < n) acc = sub_cmul(acc, F[p][i], x[p]);
                x[i] = rounded(cscale(acc, inv[i]));
                g[i] = x[i];
            }
        } else {
            if (n > 0) {
                double dmax = 0.0;
                for (int i = 0; i < n; ++i) dmax = G[i][i].x > dmax ? G[i][i].x : dmax;
                for (int i = 0; i < n; ++i) {
                    double d = G[i][i].x;
                    for (int p = 0; p < i; ++p) d -= cabs2(Lm[i][p]);
                    if (!(d > CHOL_REL * dmax)) {
                        kok = i;
                        break;
                    }
                    const double dd = sqrt(d);
                    Lm[i][i] = d2(dd, 0.0);
                    for (int r = i + 1; r < n; ++r) {
                        double2 acc = G[r][i];
                        for (int p = 0; p < i; ++p) acc = csub(acc, cmul(Lm[r][p], cconj(Lm[i][p])));
                        Lm[r][i] = cscale(acc, 1.0 / dd);
                    }
                }
            }
            n = kok;
            for (int i = 0; i < n; ++i) {
                double2 acc = cvec[i];
                for (int p = 0; p < i; ++p) acc = csub(acc, cmul(Lm[i][p], zz[p]));
                zz[i] = cscale(acc, 1.0 / Lm[i][i].x);
            }
            for (int i = n - 1; i >= 0; --i) {
                double2 acc = zz[i];
                for (int p = i + 1; p < n; ++p) acc = csub(acc, cmul(cconj(Lm[p][i]), g[p]));
                g[i] = cscale(acc, 1.0 / Lm[i][i].x);
            }
        }
        for (int i = n; i < LMAX; ++i) g[i] = d2(0, 0);
        for (int i = 0; i < LMAX; ++i) S.gam[i] = g[i];
        S.l_mr = n;
        lmr_sh = n;
        if (L >= 1) S.dots += L * (L + 3) / 2;
        if (!S.exhausted) {
            if (n < l) S.broken = 1;
            if (n == l) S.omega = g[l - 1];
        }
        if (a.record && S.m < S.max_outer) {
            for (int i = 0; i < LMAX; ++i) a.tape_gam[((size_t)rhs * S.max_outer + S.m) * LMAX + i] = g[i];
        }
    }
    __syncthreads();
    const int lm = lmr_sh;
    for (int q = threadIdx.x; q < S.nact; q += BLOCK) {
        const int s = S.act[q];
        ShiftState &H = st.H[s];
        MRCoef &c = a.mc[(size_t)rhs * NSMAX + q];
        c.s = s;
        for (int k = 0; k < LMAX; ++k) c.kc[k] = d2(0, 0);
        c.inv_q = d2(1, 0);
        if (!H.active || lm == 0) {
            c.live = 0;
            continue;
        }
        const double sp = H.sp;
        double2 qs = d2(1, 0);
        double qterms = 1.0;
        double p = 1.0;   // (-sp)^i
        for (int i = 1; i <= lm; ++i) {
            p *= -sp;
            const double2 t = cmul(g[i - 1], d2(p, 0.0));
            qs = csub(qs, t);
            qterms += cmod(t);
        }
        const bool brk = !cfinite(qs) || cmod(qs) < ZETA_MIN || cmod(qs) <= BREAK_REL * qterms;
        if (brk || !(cmod(H.zeta) * cmod(H.psi) * cmod(qs) <= ZETA_MAX)) {
            H.active = 0;
            H.broken = brk ? 1 : 0;
            H.stopped = 1;
            H.iters = S.m;
            c.live = 0;
            continue;
        }
        const double2 inv_q = cdiv(d2(1, 0), qs);
        const double2 kap = cdiv(d2(1, 0), cmul(H.zeta, H.psi));
        // kappa sum_i g_i (-sp)^(i - 1 - k) / q, i = k + 1..lm
        for (int k = 0; k < lm; ++k) {
            double2 acc = d2(0, 0);
            double p = 1.0;
            for (int i = k + 1; i <= lm; ++i) {
                acc = cadd(acc, cmul(g[i - 1], d2(p, 0.0)));
                p *= -sp;
            }
            c.kc[k] = cmul(kap, cmul(acc, inv_q));
        }
        c.inv_q = inv_q;
        c.live = 1;
        H.psi = cmul(H.psi, qs);
    }
}

// Mixed precision: decide whether the outer iteration ends with a reliable
// update r_0 = b - S x (FP64): when ||r_0|| has dropped below 0.1 of its
// largest value since the last one, when any shift would freeze on the
// recursively updated residual, or when the Krylov space looks exhausted.
template <int NT>
__device__ __forceinline__ void sc_rel_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    if (NT == BLOCK && (!S.run || !S.mixed)) return;
    const double r02 = sum1<NT>(prow(a, rhs) + 2 * a.ps, a.nblk);
    st.arrive();
    if (NT != BLOCK && (!S.run || !S.mixed)) return;
    if (threadIdx.x >= 64) return;
    const double rn = sqrt(r02);
    bool due = false;
    if ((int)threadIdx.x < S.nact) {
        const ShiftState &H = st.H[S.act[threadIdx.x]];
        if (H.active)
            due = S.forced ? (S.m + 1 >= H.force)
                           : (rn / (cmod(cmul(H.zeta, H.psi)) * S.bnorm) <= FREEZE_FRAC * S.tol);
    }
    const bool freeze = __any(due);
    if (threadIdx.x != 0) return;
    if (rn > S.rmax) S.rmax = rn;
    S.rel = (rn <= 0.1 * S.rmax || freeze || S.exhausted) ? 1 : 0;
}

template <int NT>
__device__ __forceinline__ void sc_conv_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    if (NT == BLOCK && !S.run) return;
    const double *row = prow(a, rhs);
    double re, im, r02;
    sum3<NT>(row, a.ps, a.nblk, re, im, r02);
    st.arrive();
    if (NT != BLOCK && !S.run) return;
    __shared__ double rn;
    if (threadIdx.x == 0) {
        rn = sqrt(r02);
        S.rnorm0 = rn;
        S.rho1 = d2(re, im);
        if (a.record && S.m < S.max_outer) {
            TapeOuter &o = a.tape_outer[(size_t)rhs * S.max_outer + S.m];
            o.l_eff = S.l_eff;
            o.l_mr = S.exhausted ? 0 : S.l_mr;
            o.partial = S.partial;
            o.exhausted = S.exhausted;
            o.rel = S.rel;
        }
        if (S.rel) {
            S.reliable += 1;
            S.rmax = rn;
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < S.nact; q += BLOCK) {
        ShiftState &H = st.H[S.act[q]];
        if (!H.active) continue;
        const double res = rn / (cmod(cmul(H.zeta, H.psi)) * S.bnorm);
        H.res = res;
        bool done = S.forced ? (S.m + 1 >= H.force) : (res <= FREEZE_FRAC * S.tol);
        // an exhausted Krylov space ends the solve; in mixed precision the
        // residual was just recomputed in FP64, so a shift that still misses
        // its tolerance is reported as not converged
        if (S.exhausted && !S.mixed) done = true;
        if (done) {
            H.active = 0;
            H.iters = S.m + 1;
        }
    }
    __syncthreads();
    // the shifts still active, in their order: a shift per lane of wavefront 0
    if (threadIdx.x >= 64) return;
    const int s = threadIdx.x;
    bool live = false, brk = false;
    if (s < S.nshift) {
        const ShiftState &H = st.H[s];
        live = H.active;
        brk = H.broken;
    }
    const unsigned long long lv = __ballot(live);
    const int nact = __popcll(lv);
    const bool anybroken = __any(brk);
    if (live) S.act[__popcll(lv & ((1ull << s) - 1ull))] = s;
    const bool ends = S.broken || S.exhausted || (S.m + 1 >= S.max_outer);
    if (live && ends) st.H[s].iters = S.m + 1;
    if (threadIdx.x == 0) {
        S.nact = nact;
        S.m += 1;
        S.rel = 0;
        if (nact == 0 || ends) {
            S.run = 0;
            if (nact > 0) {
                S.status = S.broken ? S_BREAKDOWN : S_NOT_CONVERGED;
            } else {
                S.status = anybroken ? S_BREAKDOWN : S_OK;
            }
        }
        S.bicg_on = 1;
        S.l_eff = 0;
        S.l_mr = 0;
        S.partial = 0;
        for (int i = 0; i < LMAX; ++i) S.step_flag[i] = 0;
        // the next outer iteration's first beta reads the sums this stage took
        if (a.then_beta && S.run) beta_step(a, S, rhs, 0, d2(re, im), r02);
    }
}

// Deferred single pass: every active shift's update over the outer iteration
// that just ended, as coefficients on the iteration's basis (see DeferCoef):
// the seed's r_i, u_i exactly as the vector kernels updated them (the recorded
// beta, alpha and step flags), and the shift's u^s_i and x^s increment by the
// recurrences of the per-step form (the recorded step coefficients of every
// step and the MR coefficients).  Vectors no step defined are zero, as the
// per-step form multiplies their stale contents by zero coefficients.  The
// recurrences act on each basis index alone: one work-item per (shift, index)
// with its column of each in registers.  One work-item per shift, its arrays
// in scratch memory, took 107 us a launch at l = 4 with 16 shifts.
template <int L>
__device__ __forceinline__ void sc_defer_body(const ScalarArgs &a, int rhs, const SeedState &S) {
    if (!S.run) return;
    constexpr int nb = 2 * L + 2, self = nb;
    for (int item = threadIdx.x; item < S.nact * NDEF; item += blockDim.x) {
        const int q = item / NDEF, b = item - q * NDEF;
        DeferCoef &d = a.dc[(size_t)rhs * NSMAX + q];
        if (b == 0) {
            d.s = S.act[q];
            d.live = 1;
        }
        if (b > nb) {
            d.cu[b] = d.cx[b] = d2(0, 0);
            continue;
        }
        double2 R[L + 1], U[L + 1], w[L + 1], dx = d2(0, 0);
#pragma unroll
        for (int i = 0; i <= L; ++i) R[i] = U[i] = w[i] = d2(0, 0);
        if (b == 0) R[0] = d2(1, 0);
        if (b == 1) U[0] = d2(1, 0);
        if (b == self) w[0] = d2(1, 0);
        bool live = true, on = true;   // on: the iteration's steps have not ended
#pragma unroll
        for (int j = 0; j < L; ++j) {
            const int flag = on ? S.step_flag[j] : 0;
            if (flag == 0) {
                on = false;
                continue;
            }
            const double2 beta = S.step_beta[j];
#pragma unroll
            for (int i = 0; i <= j; ++i) U[i] = csub(R[i], cmul(beta, U[i]));
            U[j + 1] = b == 2 + 2 * j ? d2(1, 0) : d2(0, 0);
            if (flag == 1) {
                on = false;
                continue;
            }
            const StepCoef &c = a.sc_hist[((size_t)rhs * LMAX + j) * NSMAX + q];
            if (live && c.live) {
#pragma unroll
                for (int i = 0; i <= j; ++i) w[i] = csub(cmul(c.kap, R[i]), cmul(c.beta_s, w[i]));
                dx = cfma(c.alpha_s, w[0], dx);
                w[j + 1] = csub(cadd(cmul(c.a1, R[j]), cmul(c.a2, U[j + 1])), cscale(w[j], c.sp));
            } else {
                live = false;
            }
            const double2 alpha = S.step_alpha[j];
#pragma unroll
            for (int i = 0; i <= j; ++i) R[i] = csub(R[i], cmul(alpha, U[i + 1]));
            R[j + 1] = b == 3 + 2 * j ? d2(1, 0) : d2(0, 0);
        }
        const MRCoef &m = a.mc[(size_t)rhs * NSMAX + q];
        if (live && m.live) {
#pragma unroll
            for (int k = 0; k < L; ++k) dx = cfma(m.kc[k], R[k], dx);
            double2 u0 = w[0];
#pragma unroll
            for (int i = 1; i <= L; ++i) u0 = csub(u0, cmul(S.gam[i - 1], w[i]));
            w[0] = cmul(u0, m.inv_q);
        }
        // a shift whose recurrences stopped this iteration keeps the part
        // applied before: the per-step form updated it until then
        d.cu[b] = w[0];
        d.cx[b] = dx;
    }
}

// The seed's step recurrences of this outer iteration (the steps it completed,
// step_flag), replayed on the coefficients of its basis: r_i and u_i as sums
// over B (see SeedBasis), R[i][b] and U[i][b].  Steps in the order and with
// the arithmetic of the explicit form: u_i = r_i - beta u_i (i <= j),
// u_{j+1} = S u_j, then r_i = r_i - alpha u_{i+1} (i <= j), r_{j+1} = S r_j.
// The recurrences act on each basis index b alone: one work-item per b
// (column b of R and U).
// STEP(j, flag, beta, alpha) gives step j's flag and coefficients.
template <typename STEP>
__device__ inline void basis_replay_col(const STEP &step, int l, int b, double2 (*R)[NBB], double2 (*U)[NBB]) {
    for (int i = 0; i <= l; ++i) R[i][b] = U[i][b] = d2(0, 0);
    if (b == 0) R[0][0] = d2(1, 0);
    if (b == 1) U[0][1] = d2(1, 0);
    for (int j = 0; j < l; ++j) {
        int flag;
        double2 beta, alpha;
        step(j, flag, beta, alpha);
        if (flag == 0) break;
        for (int i = 0; i <= j; ++i) U[i][b] = csub(R[i][b], cmul(beta, U[i][b]));
        if (b == 2 + 2 * j) U[j + 1][b] = d2(1, 0);
        if (flag == 1) break;
        for (int i = 0; i <= j; ++i) R[i][b] = csub(R[i][b], cmul(alpha, U[i + 1][b]));
        if (b == 3 + 2 * j) R[j + 1][b] = d2(1, 0);
    }
}
__device__ inline void seed_basis_replay_col(const SeedState &S, int l, int b, double2 (*R)[NBB],
                                             double2 (*U)[NBB]) {
    basis_replay_col(
        [&](int j, int &flag, double2 &beta, double2 &alpha) {
            flag = S.step_flag[j];
            beta = S.step_beta[j];
            alpha = S.step_alpha[j];
        },
        l, b, R, U);
}

// Basis form, before the MR step: every r_i and u_i of the outer iteration as
// coefficients on its basis.
__device__ __forceinline__ void sc_basis_body(const ScalarArgs &a, int rhs, const SeedState &S) {
    if (!S.run) return;
    __shared__ double2 R[LMAX + 1][NBB], U[LMAX + 1][NBB];
    const int b = threadIdx.x;
    if (b >= NBB) return;
    seed_basis_replay_col(S, a.l, b, R, U);
    SeedBasis &B = a.sb[rhs];
    for (int i = 0; i <= LMAX; ++i) {
        B.r[i][b] = i <= a.l ? R[i][b] : d2(0, 0);
        B.u[i][b] = i <= a.l ? U[i][b] : d2(0, 0);
    }
}

// Basis form with a sparse r~, after the MR step's coefficients and before
// the MR update overwrites r_0 and u_0: r_0 after the MR step at the list's
// entries (the MR update's combined coefficients), <r~, r_0>, and the next
// outer iteration's beta = alpha rho_1 / rho_0 with rho_0 <- -omega rho_0
// (as its first step will find it), into S (one block per rhs).
template <int L>
__device__ __forceinline__ void basis_spec_body(const BasisArgs<double> &a, int rhs, SeedState &S) {
    if (!S.run) return;
    constexpr int NBL = 2 * L + 2;
    __shared__ double2 c_r[NBL];
    __shared__ double2 rk[SPARSE_MAX];
    if (threadIdx.x < NBL) {
        const int b = threadIdx.x;
        const SeedBasis &SB = a.sb[rhs];
        const int lm = S.l_mr < L ? S.l_mr : L;
        double2 vr = SB.r[0][b];
        for (int i = 1; i <= lm; ++i) vr = csub(vr, cmul(S.gam[i - 1], SB.r[i][b]));
        c_r[b] = vr;
    }
    __syncthreads();
    const int nbu = basis_used(S);
    const int nk = a.sp_cnt[rhs];
    if ((int)threadIdx.x < nk) {
        const long e = a.sp_idx[(size_t)rhs * a.sp_max + threadIdx.x];
        double2 r0 = d2(0, 0);
        for (int b = 0; b < nbu; ++b) r0 = cfma(c_r[b], bvec(a, b, rhs, e), r0);
        rk[threadIdx.x] = r0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double p0 = 0.0, p1 = 0.0;
        for (int k = 0; k < nk; ++k) {
            const double2 t = a.sp_val[(size_t)rhs * a.sp_max + k], o = rk[k];
            p0 += t.x * o.x + t.y * o.y;
            p1 += t.x * o.y - t.y * o.x;
        }
        const double2 rho0 = cneg(cmul(S.omega, S.rho0));
        S.spec_rho1 = d2(p0, p1);
        S.beta_spec = cdiv(cmul(S.alpha, d2(p0, p1)), rho0);
    }
}

// Replay of the double pass in basis form, after outer iteration m's steps:
// the recorded steps replayed on the basis coefficients, then the recorded
// MR step, r_0 - sum_i gamma_i r_i and u_0 - sum_i gamma_i u_i (i <= lm),
// with the arithmetic of the first pass's MR update.
__device__ __forceinline__ void sc_basis_replay_body(const BasisReplayArgs &a, int rhs) {
    __shared__ double2 R[LMAX + 1][NBB], U[LMAX + 1][NBB];
    const ReplayStep *rs = a.rs + ((size_t)rhs * a.Mcap + a.m) * a.l;
    const ReplayOuter &ro = a.ro[(size_t)rhs * a.Mcap + a.m];
    const int b = threadIdx.x;
    if (b >= NBB) return;
    basis_replay_col(
        [&](int j, int &flag, double2 &beta, double2 &alpha) {
            flag = rs[j].flag;
            beta = rs[j].beta;
            alpha = rs[j].alpha;
        },
        a.l, b, R, U);
    const int lm = ro.lm < a.l ? ro.lm : a.l;
    double2 vr = R[0][b], vu = U[0][b];
    for (int i = 1; i <= lm; ++i) {
        vr = csub(vr, cmul(ro.gam[i - 1], R[i][b]));
        vu = csub(vu, cmul(ro.gam[i - 1], U[i][b]));
    }
    SeedBasis &B = a.sb[rhs];
    B.r[0][b] = vr;
    B.u[0][b] = vu;
    if (b == 0) {
        int le = 0;
        while (le < a.l && rs[le].flag == 2) ++le;
        B.nbu = (rs[0].flag == 0 && ro.lm == 0) ? 0 : 2 * le + 2;
    }
}

// Basis form, before step j >= 1: could the exhaustion test of this step
// fire?  It reads ||r_0|| after step j-1, which the basis form does not
// form; but then r_{j-1} = S^(j-1) r_0 (the steps keep r_{i+1} = S r_i), so
// ||r_0|| >= ||r_{j-1}|| / ||S||^(j-1), with norm_a an upper bound of ||S||.
// Where ||r_{j-1}|| (partial row 4, from the step's r-update) is within
// twice that factor of the test's threshold, exh_check is set and r_0's
// coefficients are written for the kernel that forms it; otherwise the test
// cannot fire and is left out.
template <int NT>
__device__ __forceinline__ void sc_exh_body(const ScalarArgs &a, int rhs, StageState<NT> &st) {
    SeedState &S = st.S;
    const int j = a.j;
    const double *row = prow(a, rhs);
    const double rj1 = sqrt(sum1<NT>(row + 4 * a.ps, a.nblk2));
    st.arrive();
    if (!S.run || !S.bicg_on) {
        if (threadIdx.x == 0) S.exh_check = 0;
        return;
    }
    __shared__ int check;
    __shared__ double2 R[LMAX + 1][NBB], U[LMAX + 1][NBB];
    const bool test = !S.forced && S.nact > 0;
    const double mn = (threadIdx.x < 64 && test) ? min_shift_scale(S, st.H) : 0.0;
    if (threadIdx.x == 0) {
        check = 0;
        if (test) {
            double fac = 2.0;
            for (int k = 0; k < j - 1; ++k) fac *= a.norm_a;
            if (rj1 <= fac * FREEZE_FRAC * S.tol * S.bnorm * mn) check = 1;
        }
        S.exh_check = check;
    }
    __syncthreads();
    if (!check) return;
    const int b = threadIdx.x;
    if (b >= NBB) return;
    seed_basis_replay_col(S, a.l, b, R, U);
    a.sb[rhs].r[0][b] = R[0][b];
}

}  // namespace dev
}  // namespace msb
