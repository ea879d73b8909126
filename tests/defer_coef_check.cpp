// The deferred single pass's coefficients (sc_defer_body) on the CPU, for
// every l and up to 64 shifts, against the recurrences of the per-step form
// written out on whole coefficient vectors in long double.  The difference is
// measured in units of the rounding of the terms: the same recurrences on
// absolute values.  Prints the largest one per l.
#include <algorithm>
#include <complex>
#include <cstdio>
#include <random>
#include <vector>

#include "scalar_dev.h"

#include "emu/block_emu.h"

using namespace msb;
typedef std::complex<long double> Z;
static Z z(double2 a) { return Z(a.x, a.y); }

// flags: the iteration's steps (2 full, 1 ended after its u-Mv, 0 none)
template <int L>
static double check(std::mt19937 &rng, int nact, const std::vector<int> &flags, int dead) {
    std::normal_distribution<double> g;
    auto c = [&] { return d2(g(rng), g(rng)); };
    SeedState S;
    std::memset(&S, 0, sizeof(S));
    S.run = 1;
    S.nact = nact;
    for (int q = 0; q < nact; ++q) S.act[q] = (q * 37 + 11) % NSMAX;
    for (int j = 0; j < L; ++j) {
        S.step_flag[j] = flags[j];
        S.step_beta[j] = c();
        S.step_alpha[j] = c();
        S.gam[j] = c();
    }
    std::vector<StepCoef> hist((size_t)LMAX * NSMAX);
    std::vector<MRCoef> mc(NSMAX);
    std::vector<DeferCoef> dc(NSMAX);
    for (int q = 0; q < nact; ++q) {
        for (int j = 0; j < L; ++j) {
            StepCoef &s = hist[(size_t)j * NSMAX + q];
            s.kap = c(), s.beta_s = c(), s.alpha_s = c(), s.a1 = c(), s.a2 = c();
            s.sp = std::fabs(g(rng));
            s.live = !(q == dead && j >= 1);
        }
        for (int k = 0; k < LMAX; ++k) mc[q].kc[k] = k < L ? c() : d2(0, 0);
        mc[q].inv_q = c();
        mc[q].live = q != dead;
    }
    ScalarArgs a;
    a.sc_hist = hist.data();
    a.mc = mc.data();
    a.dc = dc.data();
    a.l = L;
    std::vector<int> waves;
    for (int w = 0; w < 8; ++w) waves.push_back(w);
    const std::string f = emu::run_block(512, waves.data(), [&] { dev::sc_defer_body<L>(a, 0, S); });
    if (!f.empty()) return INFINITY;
    constexpr int nb = 2 * L + 2;
    double worst = 0;
    for (int q = 0; q < nact; ++q) {
        // the recurrences, and the same on absolute values
        Z R[L + 1][NDEF] = {}, U[L + 1][NDEF] = {}, w[L + 1][NDEF] = {}, dx[NDEF] = {};
        long double aR[L + 1][NDEF] = {}, aU[L + 1][NDEF] = {}, aw[L + 1][NDEF] = {}, ax[NDEF] = {};
        R[0][0] = U[0][1] = w[0][nb] = 1;
        aR[0][0] = aU[0][1] = aw[0][nb] = 1;
        bool live = true;
        for (int j = 0; j < L && flags[j]; ++j) {
            const Z be = z(S.step_beta[j]), al = z(S.step_alpha[j]);
            for (int b = 0; b <= nb; ++b)
                for (int i = 0; i <= j; ++i) {
                    U[i][b] = R[i][b] - be * U[i][b];
                    aU[i][b] = aR[i][b] + std::abs(be) * aU[i][b];
                }
            U[j + 1][2 + 2 * j] = 1;
            aU[j + 1][2 + 2 * j] = 1;
            if (flags[j] == 1) break;
            const StepCoef &s = hist[(size_t)j * NSMAX + q];
            live = live && s.live;
            for (int b = 0; b <= nb && live; ++b) {
                for (int i = 0; i <= j; ++i) {
                    w[i][b] = z(s.kap) * R[i][b] - z(s.beta_s) * w[i][b];
                    aw[i][b] = std::abs(z(s.kap)) * aR[i][b] + std::abs(z(s.beta_s)) * aw[i][b];
                }
                dx[b] += z(s.alpha_s) * w[0][b];
                ax[b] += std::abs(z(s.alpha_s)) * aw[0][b];
                w[j + 1][b] = z(s.a1) * R[j][b] + z(s.a2) * U[j + 1][b] - (long double)s.sp * w[j][b];
                aw[j + 1][b] = std::abs(z(s.a1)) * aR[j][b] + std::abs(z(s.a2)) * aU[j + 1][b] + s.sp * aw[j][b];
            }
            for (int b = 0; b <= nb; ++b)
                for (int i = 0; i <= j; ++i) {
                    R[i][b] -= al * U[i + 1][b];
                    aR[i][b] += std::abs(al) * aU[i + 1][b];
                }
            R[j + 1][3 + 2 * j] = 1;
            aR[j + 1][3 + 2 * j] = 1;
        }
        for (int b = 0; b <= nb && live && mc[q].live; ++b) {
            for (int k = 0; k < L; ++k) {
                dx[b] += z(mc[q].kc[k]) * R[k][b];
                ax[b] += std::abs(z(mc[q].kc[k])) * aR[k][b];
            }
            for (int i = 1; i <= L; ++i) {
                w[0][b] -= z(S.gam[i - 1]) * w[i][b];
                aw[0][b] += std::abs(z(S.gam[i - 1])) * aw[i][b];
            }
            w[0][b] *= z(mc[q].inv_q);
            aw[0][b] *= std::abs(z(mc[q].inv_q));
        }
        if (dc[q].s != S.act[q] || dc[q].live != 1) return INFINITY;
        for (int b = 0; b < NDEF; ++b) {
            const Z eu = z(dc[q].cu[b]) - (b <= nb ? w[0][b] : Z(0)), ex = z(dc[q].cx[b]) - (b <= nb ? dx[b] : Z(0));
            const long double su = b <= nb ? aw[0][b] : 0, sx = b <= nb ? ax[b] : 0;
            const double u = su > 0 ? (double)(std::abs(eu) / su) : eu == Z(0) ? 0 : INFINITY;
            const double x = sx > 0 ? (double)(std::abs(ex) / sx) : ex == Z(0) ? 0 : INFINITY;
            worst = std::max(worst, std::max(u, x) / 2.220446049250313e-16);
        }
    }
    return worst;
}

template <int L>
static void all(std::mt19937 &rng) {
    double worst = 0;
    for (int nact : {1, 3, 27, 64}) {
        std::vector<int> full(L, 2);
        worst = std::max(worst, check<L>(rng, nact, full, -1));
        worst = std::max(worst, check<L>(rng, nact, full, nact / 2));
        for (int end = 0; end < L; ++end)
            for (int last : {0, 1}) {
                std::vector<int> f(L, 0);
                for (int j = 0; j < end; ++j) f[j] = 2;
                f[end] = last;
                worst = std::max(worst, check<L>(rng, nact, f, -1));
            }
    }
    std::printf("%d %.3f\n", L, worst);
}

int main() {
    std::mt19937 rng(5);
    all<1>(rng), all<2>(rng), all<3>(rng), all<4>(rng), all<5>(rng), all<6>(rng), all<7>(rng), all<8>(rng);
}
