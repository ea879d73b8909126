// Device body of the Wilson-Dirac stencil D_w(mu) (see dslash.hip for the
// operator and the epilogues): the chunked form for batches, the split form
// for small launches, and the pieces that the persistent kernel's own form
// shares with them.
#pragma once
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace msb {
namespace dev {

// multiply by one of {+1, -1, +i, -i}
template <int CODE, typename Z>
__device__ __forceinline__ Z mulcode(Z z) {
    if constexpr (CODE == 0) return z;
    else if constexpr (CODE == 1) return cneg(z);
    else if constexpr (CODE == 2) return ctimes_i(z);
    else return ctimes_mi(z);
}

// The terms of the epilogues' sums, Re and Im conj(a) b, |a|^2 and c a, with
// the multiply-add of each written out: left to the compiler, which product
// of such a sum is rounded differs between the stencil's forms.
template <typename Z>
__device__ __forceinline__ double dot_re(Z a, Z b) {
    return __builtin_fma((double)a.x, (double)b.x, (double)a.y * b.y);
}
template <typename Z>
__device__ __forceinline__ double dot_im(Z a, Z b) {
    return __builtin_fma((double)a.x, (double)b.y, -((double)a.y * b.x));
}
template <typename Z>
__device__ __forceinline__ double norm2(Z a) {
    return __builtin_fma((double)a.x, (double)a.x, (double)a.y * a.y);
}
template <typename Z>
__device__ __forceinline__ double2 ymul(Z c, Z a) {
    return d2(__builtin_fma((double)c.x, (double)a.x, -((double)c.y * a.y)),
              __builtin_fma((double)c.y, (double)a.x, (double)c.x * a.y));
}

constexpr int ONE = 0, NEG = 1, I = 2, MI = 3;

// Spin projection (1 + SGN gamma_NU) psi = (h0, h1, D2 h_Q2, D3 h_Q3) with
// h0 = psi_0 + C0 psi_P0, h1 = psi_1 + C1 psi_P1 (chiral basis).
template <int NU, int SGN> struct Proj;
template <> struct Proj<0, -1> { static constexpr int P0 = 3, C0 = I, P1 = 2, C1 = I, Q2 = 1, D2 = MI, Q3 = 0, D3 = MI; };
template <> struct Proj<0, +1> { static constexpr int P0 = 3, C0 = MI, P1 = 2, C1 = MI, Q2 = 1, D2 = I, Q3 = 0, D3 = I; };
template <> struct Proj<1, -1> { static constexpr int P0 = 3, C0 = ONE, P1 = 2, C1 = NEG, Q2 = 1, D2 = NEG, Q3 = 0, D3 = ONE; };
template <> struct Proj<1, +1> { static constexpr int P0 = 3, C0 = NEG, P1 = 2, C1 = ONE, Q2 = 1, D2 = ONE, Q3 = 0, D3 = NEG; };
template <> struct Proj<2, -1> { static constexpr int P0 = 2, C0 = I, P1 = 3, C1 = MI, Q2 = 0, D2 = MI, Q3 = 1, D3 = I; };
template <> struct Proj<2, +1> { static constexpr int P0 = 2, C0 = MI, P1 = 3, C1 = I, Q2 = 0, D2 = I, Q3 = 1, D3 = MI; };
template <> struct Proj<3, -1> { static constexpr int P0 = 2, C0 = NEG, P1 = 3, C1 = NEG, Q2 = 0, D2 = NEG, Q3 = 1, D3 = NEG; };
template <> struct Proj<3, +1> { static constexpr int P0 = 2, C0 = ONE, P1 = 3, C1 = ONE, Q2 = 0, D2 = ONE, Q3 = 1, D3 = ONE; };

// Load spin component `sp` (3 colours) of site `s`; with G5IN the lower two
// spins are negated (gamma5 applied on the fly).
template <typename T, bool G5IN>
__device__ __forceinline__ void load_spin(const C<T> *__restrict__ in, int V, int s, int sp, C<T> (&c)[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        C<T> z = in[(3 * sp + a) * V + s];
        if (G5IN && sp >= 2) z = cneg(z);
        c[a] = z;
    }
}

// acc += f * [(1 + SGN gamma_NU) reconstruction of] Umat h for a projected
// half-spinor h (h0, h1); Umat = U (DAG=false) or U^+ (DAG=true), where entry
// (a, b) of U is Ub[(3 a + b) us]: the link in global memory (us = V) or
// staged in LDS (us = CHUNK).
template <typename T, int NU, int SGN, bool DAG>
__device__ __forceinline__ void hop_h(C<T> (&acc)[4][3], const C<T> (&h)[2][3], const C<T> *__restrict__ Ub, int us,
                                      T f) {
    using P = Proj<NU, SGN>;
    C<T> g[2][3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        C<T> u0, u1, u2;
        if (!DAG) {
            u0 = Ub[(3 * a + 0) * us];
            u1 = Ub[(3 * a + 1) * us];
            u2 = Ub[(3 * a + 2) * us];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                C<T> r = cmul(u0, h[i][0]);
                r = cfma(u1, h[i][1], r);
                r = cfma(u2, h[i][2], r);
                g[i][a] = r;
            }
        } else {
            // (U^+)_{ab} = conj(U_{ba})
            u0 = Ub[(0 * 3 + a) * us];
            u1 = Ub[(1 * 3 + a) * us];
            u2 = Ub[(2 * 3 + a) * us];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                C<T> r = cmulc(u0, h[i][0]);
                r = cadd(r, cmulc(u1, h[i][1]));
                r = cadd(r, cmulc(u2, h[i][2]));
                g[i][a] = r;
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        acc[0][a] = cadd(acc[0][a], cscale(g[0][a], f));
        acc[1][a] = cadd(acc[1][a], cscale(g[1][a], f));
        acc[2][a] = cadd(acc[2][a], cscale(mulcode<P::D2>(g[P::Q2][a]), f));
        acc[3][a] = cadd(acc[3][a], cscale(mulcode<P::D3>(g[P::Q3][a]), f));
    }
}

// acc += f * (1 + SGN gamma_NU) Umat psi(sn), psi loaded here (one spin at a
// time; used by the persistent kernel's stencil).
template <typename T, int NU, int SGN, bool DAG, bool G5IN>
__device__ __forceinline__ void hop(C<T> (&acc)[4][3], const C<T> *__restrict__ in,
                                   const C<T> *__restrict__ Ub, int us, int V, int sn, T f) {
    using P = Proj<NU, SGN>;
    C<T> h[2][3];
    {
        C<T> p0[3], p1[3], q0[3], q1[3];
        load_spin<T, G5IN>(in, V, sn, 0, p0);
        load_spin<T, G5IN>(in, V, sn, 1, p1);
        load_spin<T, G5IN>(in, V, sn, P::P0, q0);
        load_spin<T, G5IN>(in, V, sn, P::P1, q1);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            h[0][a] = cadd(p0[a], mulcode<P::C0>(q0[a]));
            h[1][a] = cadd(p1[a], mulcode<P::C1>(q1[a]));
        }
    }
    hop_h<T, NU, SGN, DAG>(acc, h, Ub, us, f);
}

// Element k (= 3 spin + colour) of site s: base in + k V is the same for the
// whole wavefront and the site offset is a 32-bit unsigned index, so each
// component load takes a scalar base and one vector offset per site.
template <typename E>
__device__ __forceinline__ E &elem(E *__restrict__ p, int k, int V, int s) {
    return (p + (size_t)k * (unsigned)V)[(unsigned)s];
}
// An operand the chunked form reads once per sweep (v, w, r~, y): streamed
// past L2, like its output, so that it does not evict neighbour spinors.
template <typename E>
__device__ __forceinline__ E ld_stream(const E *__restrict__ p, int k, int V, int s) {
    const E &q = elem(p, k, V, s);
    E r;
    r.x = __builtin_nontemporal_load(&q.x);
    r.y = __builtin_nontemporal_load(&q.y);
    return r;
}

// The 12 components of psi(s) ([gamma5] applied: lower spins negated).
template <typename T, bool G5IN>
__device__ __forceinline__ void load_site(const C<T> *__restrict__ in, int V, int s, C<T> (&b)[12]) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        C<T> z = elem(in, k, V, s);
        if (G5IN && k >= 6) z = cneg(z);
        b[k] = z;
    }
}

// h = the two independent spins of (1 + SGN gamma_NU) psi
template <typename T, int NU, int SGN>
__device__ __forceinline__ void project(const C<T> (&b)[12], C<T> (&h)[2][3]) {
    using P = Proj<NU, SGN>;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        h[0][a] = cadd(b[a], mulcode<P::C0>(b[3 * P::P0 + a]));
        h[1][a] = cadd(b[3 + a], mulcode<P::C1>(b[3 * P::P1 + a]));
    }
}

// The links staged in LDS for a 64-site chunk: [8 hops][9][CHUNK].
template <typename T>
struct LdsLinks {
    const C<T> *L;
    int base;   // first site of the chunk
    __device__ __forceinline__ const C<T> *at(int nu, int bwd, int s) const {
        return L + (2 * nu + bwd) * 9 * CHUNK + (s - base);
    }
};

// Lx = 16 in the chunked form: the 16 lanes of each row of a wavefront hold
// one periodic x-line, so a site's x-neighbour values are in the lanes next
// to it.  x_rotate replaces each lane's half spinor with that of lane
// (i + 1) mod 16 (FWD) or (i - 1) mod 16 of its row (DPP row rotate), which
// is bitwise the projection the lane would have formed from the neighbour's
// loaded spinor, without its twelve loads.
template <bool FWD>
__device__ __forceinline__ int row_rot(int v) {
    return __builtin_amdgcn_update_dpp(0, v, FWD ? 0x12F : 0x121, 0xF, 0xF, false);
}
__device__ __forceinline__ double row_rot_d(double v, bool fwd) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return fwd ? __hiloint2double(row_rot<true>(hi), row_rot<true>(lo))
               : __hiloint2double(row_rot<false>(hi), row_rot<false>(lo));
}
__device__ __forceinline__ float row_rot_d(float v, bool fwd) {
    return __int_as_float(fwd ? row_rot<true>(__float_as_int(v)) : row_rot<false>(__float_as_int(v)));
}
template <typename T, bool FWD>
__device__ __forceinline__ void x_rotate(C<T> (&h)[2][3]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) h[i][c] = mk<T>(row_rot_d(h[i][c].x, FWD), row_rot_d(h[i][c].y, FWD));
}

// Order of the hop sum, chosen by the parity of z + t at the first site of
// the site's aligned 64-site group (order_parity below).  Even
// sites start from the diagonal term, -2 (4+m) psi(x), add the hops x-, x+,
// y-, y+, z-, z+, t-, t+ and scale the sum by -scale/2; odd sites add z-, z+,
// t-, t+, x-, x+, y-, y+ and form scale ((4+m) psi(x) - sum/2) at the end.
// A chunk's spinors are read by the chunk itself (its x and y hops and its
// centre) and by the z and t neighbour chunks, which have the other parity:
// an even chunk reads its own data first and then its neighbours', an odd
// chunk its neighbours' first and then its own, so co-resident chunks that
// sweep a right-hand side together read each line within a short stretch of
// the sweep, while it is still in the XCD's L2.  Every stencil form uses the
// same per-site order, so all of them give the same bits.

// The parity that picks a site's order: that of z + t at the first site of
// its aligned 64-site group.  Every form runs its wavefronts over such groups
// (chunks, and the four wavefronts of a 256-site block), so the choice is
// uniform over a wavefront and the branch on it is a scalar one: a per-lane
// choice made the waves that straddle a z-t plane (Lx Ly not a multiple of
// 64) run both orders.  Where Lx Ly is a multiple of 64 this is the site's
// own parity.
__device__ __forceinline__ int order_parity(const Geom &g, int s) {
    const int zt = (s & ~63) / (g.Lx * g.Ly);
    return __builtin_amdgcn_readfirstlane((zt % g.Lz + zt / g.Lz) & 1);
}

// m2d = -2 (4+m): acc = m2d psi(x).  No multiply-add may absorb this product
// (the forms must round it alike wherever it is inlined).
template <typename T>
__device__ __forceinline__ void diag_start_spin(C<T> (&acc)[3], const C<T> (&b)[3], T m2d) {
#pragma clang fp contract(off)
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = mk<T>(b[c].x * m2d, b[c].y * m2d);
}
template <typename T>
__device__ __forceinline__ void diag_start(C<T> (&acc)[4][3], const C<T> (&b)[12], T m2d) {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
        const C<T> bs[3] = {b[3 * sp], b[3 * sp + 1], b[3 * sp + 2]};
        diag_start_spin<T>(acc[sp], bs, m2d);
    }
}
// even sites: out = (-scale/2 [gamma5]) acc
template <typename T>
__device__ __forceinline__ void even_finish(C<T> (&acc)[4][3], T scale, int g5out) {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
        const T f = ((g5out && sp >= 2) ? (T)0.5 : (T)-0.5) * scale;
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[sp][c] = cscale(acc[sp][c], f);
    }
}
// odd sites: out = scale [gamma5] ((4+m) psi(x) - acc / 2)
template <typename T>
__device__ __forceinline__ void odd_finish_spin(C<T> (&acc)[3], const C<T> (&b)[3], T diag, T sg) {
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = cscale(csub(cscale(b[c], diag), cscale(acc[c], (T)0.5)), sg);
}
template <typename T>
__device__ __forceinline__ void odd_finish(C<T> (&acc)[4][3], const C<T> (&b)[12], T diag, T scale, int g5out) {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
        const C<T> bs[3] = {b[3 * sp], b[3 * sp + 1], b[3 * sp + 2]};
        odd_finish_spin<T>(acc[sp], bs, diag, ((g5out && sp >= 2) ? (T)-1 : (T)1) * scale);
    }
}

// The stencil and its epilogue for sites s0, s0 + sstride, ... < V of one
// right-hand side.  sstride exceeds V, so the loop body runs at most once;
// keeping it a loop with a run-time bound (and every address derived from s)
// stops the compiler from hoisting loads out of the caller's loop over
// right-hand sides.  With links in LDS the neighbours are gathered two hops
// ahead: while hop k is multiplied, the spinors of hops k + 1 and k + 2 are
// in flight (two 12-component buffers), in the parity order above.
template <typename T, int EPI, bool G5IN>
__device__ __forceinline__ void dslash_sites(const DslashArgs<T> &a, const LdsLinks<T> &lk, const C<T> *__restrict__ in,
                                             C<T> *__restrict__ out, const C<T> *__restrict__ v,
                                             const C<T> *__restrict__ rt, double2 *__restrict__ y, C<T> yc,
                                             T sig0, const C<T> *__restrict__ wsub,
                                             int s0, double (&part)[3]) {
    const int V = a.g.V;
    for (int s = s0; s < V; s += a.sstride) {
    C<T> acc[4][3];
    const int Lx = a.g.Lx, Ly = a.g.Ly, Lz = a.g.Lz, Lt = a.g.Lt;
    const int sxy = Lx * Ly, sxyz = Lx * Ly * Lz;
    const int x = s % Lx;
    const int r1 = s / Lx;
    const int yy = r1 % Ly;
    const int r2 = r1 / Ly;
    const int z = r2 % Lz;
    const int t = r2 / Lz;
    constexpr int us = CHUNK;
    const T ff = (t == Lt - 1) ? a.ef * a.bc : a.ef;
    const T fb = (t == 0) ? a.eb * a.bc : a.eb;
    const int xf = (x == Lx - 1) ? s - (Lx - 1) : s + 1;
    const int xb = (x == 0) ? s + (Lx - 1) : s - 1;
    const int yf = (yy == Ly - 1) ? s - (Ly - 1) * Lx : s + Lx;
    const int yb = (yy == 0) ? s + (Ly - 1) * Lx : s - Lx;
    const int zf = (z == Lz - 1) ? s - (Lz - 1) * sxy : s + sxy;
    const int zb = (z == 0) ? s + (Lz - 1) * sxy : s - sxy;
    const int tf = (t == Lt - 1) ? s - (Lt - 1) * sxyz : s + sxyz;
    const int tb = (t == 0) ? s + (Lt - 1) * sxyz : s - sxyz;
    C<T> bA[12], bB[12], h[2][3];
    if (order_parity(a.g, s) && Lx == 16) {
        // odd, x from the neighbouring lanes: z, t, x, y, the centre loaded
        // during the t hops and kept for the diagonal term
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[i][c] = mk<T>(0, 0);
        load_site<T, G5IN>(in, V, zf, bA);
        load_site<T, G5IN>(in, V, zb, bB);
        project<T, 2, -1>(bA, h);
        load_site<T, G5IN>(in, V, tf, bA);
        hop_h<T, 2, -1, false>(acc, h, lk.at(2, 0, s), us, (T)1);
        project<T, 2, +1>(bB, h);
        load_site<T, G5IN>(in, V, tb, bB);
        hop_h<T, 2, +1, true>(acc, h, lk.at(2, 1, s), us, (T)1);
        project<T, 3, -1>(bA, h);
        load_site<T, G5IN>(in, V, s, bA);    // the centre
        hop_h<T, 3, -1, false>(acc, h, lk.at(3, 0, s), us, ff);
        project<T, 3, +1>(bB, h);
        load_site<T, G5IN>(in, V, yf, bB);
        hop_h<T, 3, +1, true>(acc, h, lk.at(3, 1, s), us, fb);
        project<T, 0, -1>(bA, h);
        x_rotate<T, true>(h);
        hop_h<T, 0, -1, false>(acc, h, lk.at(0, 0, s), us, (T)1);
        project<T, 0, +1>(bA, h);
        x_rotate<T, false>(h);
        hop_h<T, 0, +1, true>(acc, h, lk.at(0, 1, s), us, (T)1);
        project<T, 1, -1>(bB, h);
        load_site<T, G5IN>(in, V, yb, bB);
        hop_h<T, 1, -1, false>(acc, h, lk.at(1, 0, s), us, (T)1);
        project<T, 1, +1>(bB, h);
        hop_h<T, 1, +1, true>(acc, h, lk.at(1, 1, s), us, (T)1);
        odd_finish<T>(acc, bA, a.diag, a.scale, a.g5out);
    } else if (order_parity(a.g, s)) {
        // odd: z, t, x, y, then the centre
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[i][c] = mk<T>(0, 0);
        load_site<T, G5IN>(in, V, zf, bA);
        load_site<T, G5IN>(in, V, zb, bB);
        project<T, 2, -1>(bA, h);
        load_site<T, G5IN>(in, V, tf, bA);
        hop_h<T, 2, -1, false>(acc, h, lk.at(2, 0, s), us, (T)1);
        project<T, 2, +1>(bB, h);
        load_site<T, G5IN>(in, V, tb, bB);
        hop_h<T, 2, +1, true>(acc, h, lk.at(2, 1, s), us, (T)1);
        project<T, 3, -1>(bA, h);
        load_site<T, G5IN>(in, V, xf, bA);
        hop_h<T, 3, -1, false>(acc, h, lk.at(3, 0, s), us, ff);
        project<T, 3, +1>(bB, h);
        load_site<T, G5IN>(in, V, xb, bB);
        hop_h<T, 3, +1, true>(acc, h, lk.at(3, 1, s), us, fb);
        project<T, 0, -1>(bA, h);
        load_site<T, G5IN>(in, V, yf, bA);
        hop_h<T, 0, -1, false>(acc, h, lk.at(0, 0, s), us, (T)1);
        project<T, 0, +1>(bB, h);
        load_site<T, G5IN>(in, V, yb, bB);
        hop_h<T, 0, +1, true>(acc, h, lk.at(0, 1, s), us, (T)1);
        project<T, 1, -1>(bA, h);
        load_site<T, G5IN>(in, V, s, bA);    // the centre, for the diagonal term
        hop_h<T, 1, -1, false>(acc, h, lk.at(1, 0, s), us, (T)1);
        project<T, 1, +1>(bB, h);
        hop_h<T, 1, +1, true>(acc, h, lk.at(1, 1, s), us, (T)1);
        odd_finish<T>(acc, bA, a.diag, a.scale, a.g5out);
    } else {
        // even: the centre, x, y, z, t
        if (Lx == 16) {
            // x from the neighbouring lanes (the centre's projections)
            load_site<T, G5IN>(in, V, s, bB);
            load_site<T, G5IN>(in, V, yf, bA);
            diag_start<T>(acc, bB, (T)-2 * a.diag);
            project<T, 0, -1>(bB, h);
            x_rotate<T, true>(h);
            hop_h<T, 0, -1, false>(acc, h, lk.at(0, 0, s), us, (T)1);
            project<T, 0, +1>(bB, h);
            load_site<T, G5IN>(in, V, yb, bB);
            x_rotate<T, false>(h);
            hop_h<T, 0, +1, true>(acc, h, lk.at(0, 1, s), us, (T)1);
        } else {
            C<T> cc[12];
            load_site<T, G5IN>(in, V, s, cc);
            load_site<T, G5IN>(in, V, xf, bA);
            load_site<T, G5IN>(in, V, xb, bB);
            diag_start<T>(acc, cc, (T)-2 * a.diag);
            project<T, 0, -1>(bA, h);
            load_site<T, G5IN>(in, V, yf, bA);
            hop_h<T, 0, -1, false>(acc, h, lk.at(0, 0, s), us, (T)1);
            project<T, 0, +1>(bB, h);
            load_site<T, G5IN>(in, V, yb, bB);
            hop_h<T, 0, +1, true>(acc, h, lk.at(0, 1, s), us, (T)1);
        }
        project<T, 1, -1>(bA, h);
        load_site<T, G5IN>(in, V, zf, bA);
        hop_h<T, 1, -1, false>(acc, h, lk.at(1, 0, s), us, (T)1);
        project<T, 1, +1>(bB, h);
        load_site<T, G5IN>(in, V, zb, bB);
        hop_h<T, 1, +1, true>(acc, h, lk.at(1, 1, s), us, (T)1);
        project<T, 2, -1>(bA, h);
        load_site<T, G5IN>(in, V, tf, bA);
        hop_h<T, 2, -1, false>(acc, h, lk.at(2, 0, s), us, (T)1);
        project<T, 2, +1>(bB, h);
        load_site<T, G5IN>(in, V, tb, bB);
        hop_h<T, 2, +1, true>(acc, h, lk.at(2, 1, s), us, (T)1);
        project<T, 3, -1>(bA, h);
        hop_h<T, 3, -1, false>(acc, h, lk.at(3, 0, s), us, ff);
        project<T, 3, +1>(bB, h);
        hop_h<T, 3, +1, true>(acc, h, lk.at(3, 1, s), us, fb);
        even_finish<T>(acc, a.scale, a.g5out);
    }
#pragma unroll
    for (int sp = 0; sp < 4; ++sp) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int k = 3 * sp + c;
            C<T> o = acc[sp][c];
            C<T> vk;
            if (EPI != EPI_PLAIN) {
                vk = ld_stream(v, k, V, s);
                o = cadd(o, cscale(vk, sig0));
            }
            if (EPI == EPI_SV2) o = csub(o, ld_stream(wsub, k, V, s));
            // streamed past L2: the output is not read again by this sweep,
            // and its lines would evict neighbour spinors
            C<T> &d = elem(out, k, V, s);
            __builtin_nontemporal_store(o.x, &d.x);
            __builtin_nontemporal_store(o.y, &d.y);
            if (EPI == EPI_MV) {
                const C<T> r = ld_stream(rt, k, V, s);
                part[0] += dot_re(r, o);
                part[1] += dot_im(r, o);
            }
            if (EPI == EPI_MVV) part[0] += dot_re(vk, o);
            // EPI_MVN: no r~ here, its dot comes from a sparse list
            else if (epi_dots(EPI)) part[2] += norm2(o);
            if (EPI == EPI_MV_Y) {
                double2 &yr = elem(y, k, V, s);
                double2 yv = ld_stream(y, k, V, s);
                yv = cadd(yv, ymul(yc, o));
                __builtin_nontemporal_store(yv.x, &yr.x);
                __builtin_nontemporal_store(yv.y, &yr.y);
            }
        }
    }
    }
}

// Operand pointers of right-hand side rhs.
template <typename T>
struct RhsOps {
    const C<T> *in;
    C<T> *out;
    const C<T> *v, *rt;
    double2 *y;
    C<T> yc;
    T sig0;
    const C<T> *w;
};
template <typename T, int EPI>
__device__ __forceinline__ RhsOps<T> rhs_ops(const DslashArgs<T> &a, int rhs) {
    const long nv = 12L * a.g.V;
    RhsOps<T> o;
    o.in = a.in + (size_t)rhs * (a.in_rs ? a.in_rs : nv);
    o.out = a.out + (size_t)rhs * (a.out_rs ? a.out_rs : nv);
    o.v = a.v ? a.v + (size_t)rhs * (a.v_rs ? a.v_rs : nv) : nullptr;
    o.rt = a.rt ? a.rt + (size_t)rhs * (a.rt_rs ? a.rt_rs : nv) : nullptr;
    o.y = a.y ? a.y + (size_t)rhs * (a.y_rs ? a.y_rs : nv) : nullptr;
    o.yc = mk<T>(0, 0);
    if (EPI == EPI_MV_Y) o.yc = to_c<T>(ld(a.ycoef, rhs));
    o.sig0 = a.sigma0_rhs ? (T)a.sigma0_rhs[rhs] : a.sigma0;
    o.w = a.w ? a.w + (size_t)rhs * (a.w_rs ? a.w_rs : nv) : nullptr;
    return o;
}

// Site offset of the backward neighbour in direction nu.
__device__ __forceinline__ int back_neighbour(const Geom &g, int nu, int s) {
    const int d = nu == 0 ? 1 : nu == 1 ? g.Lx : nu == 2 ? g.Lx * g.Ly : g.Lx * g.Ly * g.Lz;
    const int L = nu == 0 ? g.Lx : nu == 1 ? g.Ly : nu == 2 ? g.Lz : g.Lt;
    return (s / d) % L == 0 ? s + (L - 1) * d : s - d;
}

// Chunk of a block of the chunked and the split stencil: XCD x8 owns a
// contiguous slab of chunks, walked with the time coordinate varying fastest
// (slot i of the slab) so that the t -/+ 1 neighbour planes were read moments
// earlier by the same XCD.  -1: no chunk.
template <typename T>
__device__ __forceinline__ int slab_chunk(const DslashArgs<T> &a, int x8, int i) {
    const int s0 = x8 * a.per;
    int n = a.nch - s0;
    if (n > a.per) n = a.per;
    int c = i;
    if (a.tsc) {
        const int ntl = a.per_t / a.tsc;
        const int zc = i / ntl;
        c = (i - zc * ntl) * a.tsc + zc;
    }
    return c < n ? s0 + c : -1;
}

// Chunked stencil for batches: one block of NW wavefronts per 64-site chunk
// and group of a.rpb right-hand sides (dslash_chunk_prepare says why).  The
// block first stages the chunk's eight links per site (forward U_nu(x) and
// backward U_nu(x - nu)) in LDS, then its wavefronts take the group's
// right-hand sides in turn, one site per lane, reading the links from LDS:
// the links cross the memory fabric once per chunk instead of once per
// right-hand side.  Each wavefront stages whole directions, one site per
// lane, with all 18 loads of a direction in flight and the neighbour worked
// out once; a loop over flat element indices (with two divisions and one
// exposed trip to memory per element) took 20 us of a 12-source 16^3x32
// launch (plain epilogue 226 us, now 206; 4 sources 80 us, now 64).  Which
// group a block takes varies slowest, so a launch sweeps the lattice group
// after group (one group's input and output stay nearer the caches; with the
// groups of a chunk side by side 12 sources in threes took 240 us, not 214).
template <typename T, int EPI, bool G5IN, int NW>
__device__ __forceinline__ void dslash_chunk(const DslashArgs<T> &a, int p) {
    __shared__ C<T> Ls[8 * 9 * CHUNK];
    const int i = p >> 3;
    const int grp = i / a.per_t;
    const int chunk = slab_chunk(a, p & 7, i - grp * a.per_t);
    if (chunk < 0) return;
    const int V = a.g.V;
    const int base = chunk * CHUNK;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int sl = base + lane < V ? base + lane : V - 1;   // lanes past the lattice stage its last site
    for (int nu = w; nu < 4; nu += NW) {
        const C<T> *U = a.U + (size_t)nu * 9 * (unsigned)V;
        const int sb = back_neighbour(a.g, nu, sl);
        C<T> u[18];
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            u[e] = elem(U, e, V, sl);
            u[9 + e] = elem(U, e, V, sb);
        }
#pragma unroll
        for (int e = 0; e < 18; ++e) Ls[(nu * 18 + e) * CHUNK + lane] = u[e];
    }
    __syncthreads();
    const LdsLinks<T> lk{Ls, base};
    const int r0 = grp * a.rpb, r1 = r0 + a.rpb < a.nrhs ? r0 + a.rpb : a.nrhs;
    for (int rhs = r0 + w; rhs < r1; rhs += NW) {
        if (!gate_open(a.gate, rhs)) continue;
        const RhsOps<T> o = rhs_ops<T, EPI>(a, rhs);
        double part[3] = {0.0, 0.0, 0.0};
        dslash_sites<T, EPI, G5IN>(a, lk, o.in, o.out, o.v, o.rt, o.y, o.yc, o.sig0, o.w, base + lane, part);
        double *prow = a.part + (size_t)rhs * PMAX * a.ps + chunk;
        if (EPI == EPI_MVV) {
            wave_reduce_store<1>({part[0]}, prow, a.ps);
        } else if (EPI == EPI_MVN) {
            wave_reduce_store<1>({part[2]}, prow + 2 * a.ps, a.ps);
            if (lane == 0) prow[0] = prow[a.ps] = 0.0;
        } else if (epi_dots(EPI)) {
            wave_reduce_store<3>(part, prow, a.ps);
        }
    }
}

// g = U h (U^+ h with DAG) for a link held in registers, with hop_h's
// arithmetic.
template <typename T, bool DAG>
__device__ __forceinline__ void link_mul(const C<T> (&u)[9], const C<T> (&h)[2][3], C<T> (&g)[2][3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            C<T> r;
            if (!DAG) {
                r = cmul(u[3 * a], h[i][0]);
                r = cfma(u[3 * a + 1], h[i][1], r);
                r = cfma(u[3 * a + 2], h[i][2], r);
            } else {
                r = cmulc(u[a], h[i][0]);
                r = cadd(r, cmulc(u[3 + a], h[i][1]));
                r = cadd(r, cmulc(u[6 + a], h[i][2]));
            }
            g[i][a] = r;
        }
}

// LDS of a block of the split stencil: the hops' products [8 hops][6][CHUNK]
// and, for the partials, the output and r~ (EPI_MVV: v) [12][CHUNK].
template <typename T, int EPI>
struct SplitLds {
    C<T> g[8 * 6 * CHUNK];
    C<T> o[epi_dots(EPI) ? 12 * CHUNK : 1];
    C<T> r[EPI == EPI_MV || EPI == EPI_MVV ? 12 * CHUNK : 1];
};

// The part of wavefront NU of a block of the split stencil: both hops of
// direction NU, then spin NU of the output.
template <typename T, int EPI, bool G5IN, int NU>
__device__ __forceinline__ void split_wave(const DslashArgs<T> &a, SplitLds<T, EPI> &lds, int chunk, int rhs) {
    const int lane = threadIdx.x & 63;
    const int V = a.g.V, Lt = a.g.Lt;
    const int s_ = chunk * CHUNK + lane;
    const bool valid = s_ < V;
    const int s = valid ? s_ : V - 1;   // lanes past the lattice repeat its last site and store nothing
    const int d = NU == 0 ? 1 : NU == 1 ? a.g.Lx : NU == 2 ? a.g.Lx * a.g.Ly : a.g.Lx * a.g.Ly * a.g.Lz;
    const int L = NU == 0 ? a.g.Lx : NU == 1 ? a.g.Ly : NU == 2 ? a.g.Lz : Lt;
    const int xn = NU == 3 ? s / d : (s / d) % L;
    const int sf = xn == L - 1 ? s - (L - 1) * d : s + d;
    const int sb = xn == 0 ? s + (L - 1) * d : s - d;
    const int t = NU == 3 ? xn : s / (a.g.Lx * a.g.Ly * a.g.Lz);
    const RhsOps<T> o = rhs_ops<T, EPI>(a, rhs);
    C<T> bF[12], bB[12], uF[9], uB[9];
    const C<T> *U = a.U + (size_t)NU * 9 * (unsigned)V;
    load_site<T, G5IN>(o.in, V, sf, bF);
#pragma unroll
    for (int e = 0; e < 9; ++e) uF[e] = elem(U, e, V, s);
    load_site<T, G5IN>(o.in, V, sb, bB);
#pragma unroll
    for (int e = 0; e < 9; ++e) uB[e] = elem(U, e, V, sb);
    // what spin NU's output needs besides the hops
    C<T> cen[3], vv[3], rr[3], ww[3];
    double2 yy[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int k = 3 * NU + c;
        cen[c] = elem(o.in, k, V, s);
        if (G5IN && NU >= 2) cen[c] = cneg(cen[c]);
        if (EPI != EPI_PLAIN) vv[c] = elem(o.v, k, V, s);
        if (EPI == EPI_SV2) ww[c] = elem(o.w, k, V, s);
        if (EPI == EPI_MV) rr[c] = elem(o.rt, k, V, s);
        if (EPI == EPI_MV_Y) yy[c] = elem(o.y, k, V, s);
    }
    C<T> h[2][3], gF[2][3], gB[2][3];
    project<T, NU, -1>(bF, h);
    link_mul<T, false>(uF, h, gF);
    project<T, NU, +1>(bB, h);
    link_mul<T, true>(uB, h, gB);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lds.g[((2 * NU) * 6 + 3 * i + c) * CHUNK + lane] = gF[i][c];
            lds.g[((2 * NU + 1) * 6 + 3 * i + c) * CHUNK + lane] = gB[i][c];
        }
    // r~ goes to LDS on this side of the barrier: kept in registers beyond it
    // the compiler spilled it to scratch, a vector written and read (24^3x48,
    // FP64: 238 us, now 202)
    if (EPI == EPI_MV) {
#pragma unroll
        for (int c = 0; c < 3; ++c) lds.r[(3 * NU + c) * CHUNK + lane] = rr[c];
    }
    __syncthreads();
    const T ff = (t == Lt - 1) ? a.ef * a.bc : a.ef;
    const T fb = (t == 0) ? a.eb * a.bc : a.eb;
    // acc + f * (spin NU, colour c of the hop in direction N, backward with B)
    auto add = [&](auto N_, auto B_, int c, C<T> acc) __attribute__((always_inline)) {
        constexpr int N = decltype(N_)::value, B = decltype(B_)::value;
        using P = Proj<N, B ? 1 : -1>;
        constexpr int i = NU < 2 ? NU : (NU == 2 ? P::Q2 : P::Q3);
        C<T> g = N == NU ? (B ? gB[i][c] : gF[i][c]) : lds.g[((2 * N + B) * 6 + 3 * i + c) * CHUNK + lane];
        if (NU == 2) g = mulcode<P::D2>(g);
        if (NU == 3) g = mulcode<P::D3>(g);
        return cadd(acc, cscale(g, N == 3 ? (B ? fb : ff) : (T)1));
    };
    auto both = [&](auto N_, int c, C<T> acc) __attribute__((always_inline)) {
        acc = add(N_, std::integral_constant<int, 0>{}, c, acc);
        return add(N_, std::integral_constant<int, 1>{}, c, acc);
    };
    constexpr std::integral_constant<int, 0> X{};
    constexpr std::integral_constant<int, 1> Y{};
    constexpr std::integral_constant<int, 2> Z{};
    constexpr std::integral_constant<int, 3> Ti{};
    C<T> out[3];
    if (order_parity(a.g, s)) {
#pragma unroll
        for (int c = 0; c < 3; ++c) out[c] = both(Y, c, both(X, c, both(Ti, c, both(Z, c, mk<T>(0, 0)))));
        odd_finish_spin<T>(out, cen, a.diag, ((a.g5out && NU >= 2) ? (T)-1 : (T)1) * a.scale);
    } else {
        diag_start_spin<T>(out, cen, (T)-2 * a.diag);
        const T f = ((a.g5out && NU >= 2) ? (T)0.5 : (T)-0.5) * a.scale;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            out[c] = cscale(both(Ti, c, both(Z, c, both(Y, c, both(X, c, out[c])))), f);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int k = 3 * NU + c;
        C<T> z = out[c];
        if (EPI != EPI_PLAIN) z = cadd(z, cscale(vv[c], o.sig0));
        if (EPI == EPI_SV2) z = csub(z, ww[c]);
        if (valid) elem(o.out, k, V, s) = z;
        if (EPI == EPI_MV_Y) {
            double2 yv = yy[c];
            yv = cadd(yv, ymul(o.yc, z));
            if (valid) elem(o.y, k, V, s) = yv;
        }
        if (epi_dots(EPI)) {
            lds.o[k * CHUNK + lane] = z;
            if (EPI == EPI_MVV) lds.r[k * CHUNK + lane] = vv[c];
        }
    }
    if (epi_dots(EPI)) {
        // wavefronts 0, 1, 2 sum ||out||^2, Re and Im <rt, out>: per lane over
        // the components in the other forms' order, then over the lanes
        __syncthreads();
        if (NU == 3 || (EPI == EPI_MVV && NU != 1)) return;
        constexpr int row = NU == 0 ? 2 : NU - 1;
        double x = 0.0;
        constexpr bool dots = EPI == EPI_MV || EPI == EPI_MVV;
        if ((NU == 0 || dots) && valid) {
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                const C<T> z = lds.o[k * CHUNK + lane];
                if (NU == 0) x += norm2(z);
                if constexpr (dots) {
                    const C<T> r = lds.r[k * CHUNK + lane];
                    if (NU == 1) x += dot_re(r, z);
                    if (NU == 2) x += dot_im(r, z);
                }
            }
        }
        x = wave_sum(x);
        if (lane == 0) a.part[(size_t)rhs * PMAX * a.ps + row * a.ps + chunk] = x;
    }
}

// Split stencil, for launches that cannot fill the chip with one lane per
// site (dslash_use_split): one block of four wavefronts per 64-site chunk and
// right-hand side.  A lane per site gathers its nine spinors and eight links
// in a chain of dependent trips to memory; here wavefront nu does both hops of
// direction nu, with its 24 spinor and 18 link loads and spin nu's epilogue
// operands all in flight at once, passes the products U h through LDS and
// finishes spin nu, adding the hops in the other forms' order with their
// arithmetic (the same bits).  What bounds it is one trip to memory, a barrier
// and the launch where the lattice is small, the links' traffic where it is
// large (one right-hand side moves 36 complex of links per site for 24 of
// spinor).  A lane per site against this form, FP64, one right-hand side:
// 4^3x8 9.9 -> 5.1 us, 12^3x24 17 -> 10.5, 24^3x48 (637 MB) 221 -> 155; with
// r~ and partials 11.3 -> 5.6, 19.7 -> 13.3, 262 -> 200.  Its output and
// epilogue operands use cached accesses: up to 16^3x32 the vectors of one
// right-hand side stay in the caches from one launch to the next.
template <typename T, int EPI, bool G5IN>
__device__ __forceinline__ void dslash_split(const DslashArgs<T> &a, int p) {
    __shared__ SplitLds<T, EPI> lds;
    const int i = p >> 3;
    const int slot = i / a.nrhs, rhs = i - slot * a.nrhs;
    const int chunk = slab_chunk(a, p & 7, slot);
    if (chunk < 0 || !gate_open(a.gate, rhs)) return;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w == 0) split_wave<T, EPI, G5IN, 0>(a, lds, chunk, rhs);
    else if (w == 1) split_wave<T, EPI, G5IN, 1>(a, lds, chunk, rhs);
    else if (w == 2) split_wave<T, EPI, G5IN, 2>(a, lds, chunk, rhs);
    else split_wave<T, EPI, G5IN, 3>(a, lds, chunk, rhs);
}

}  // namespace dev
}  // namespace msb
