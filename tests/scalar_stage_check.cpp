// The library's one-launch scalar stages on the CPU (tests/emu), one block
// each, over the ways a stage can end: which words of shared or device memory
// two wavefronts touch without a barrier between them, and whether all
// wavefronts meet at the same barriers.  Prints a line per run.
#include <cstdio>
#include <vector>

#include "scalar.hip"

#include "emu/block_emu.h"

using namespace msb;

namespace {
struct Call {
    std::vector<SeedState> seed;
    std::vector<ShiftState> sh;
    std::vector<StepCoef> sc, hist;
    std::vector<MRCoef> mc;
    std::vector<DeferCoef> dc;
    std::vector<SeedBasis> sb;
    std::vector<double> part;
    ScalarArgs a;
    Call(int l, bool basis)
        : seed(1), sh(NSMAX), sc(NSMAX), hist((size_t)LMAX * NSMAX), mc(NSMAX), dc(NSMAX), sb(1),
          part((size_t)PMAX * NBMAX, 1.0) {
        SeedState &S = seed[0];
        std::memset(&S, 0, sizeof(S));
        S.rho0 = S.omega = S.alpha = S.beta = S.rho1 = d2(1, 0.5);
        S.bnorm = S.rtnorm = S.rnorm0 = S.rnorm_j = S.rmax = 1.0;
        S.tol = 1e-8;
        S.run = S.bicg_on = 1;
        S.max_outer = 100;
        S.max_steps = 100 * l;
        S.nshift = S.nact = 40;
        for (int s = 0; s < NSMAX; ++s) {
            std::memset(&sh[s], 0, sizeof(ShiftState));
            sh[s].zeta = sh[s].zeta_prev = sh[s].psi = d2(1, 0);
            sh[s].sp = 0.1 * s;
            sh[s].active = s < S.nshift;
            if (s < S.nshift) S.act[s] = s;
        }
        a.seed = seed.data();
        a.sh = sh.data();
        a.sc = sc.data();
        a.sc_hist = hist.data();
        a.mc = mc.data();
        a.dc = dc.data();
        a.sb = sb.data();
        a.part = part.data();
        a.ps = NBMAX;
        a.l = l;
        a.nblk = a.nblk2 = 300;
        a.basis = basis ? 1 : 0;
        a.norm_a = 2.0;
    }
    void row(int r, double v) { std::fill(part.begin() + (size_t)r * NBMAX, part.begin() + (size_t)(r + 1) * NBMAX, v); }
};

int bad = 0;
template <typename F> void check(const char *what, int nt, const Call &start, F kernel) {
    std::vector<int> up(nt / 64), down(nt / 64);
    for (int w = 0; w < nt / 64; ++w) up[w] = down[nt / 64 - 1 - w] = w;
    SeedState first;
    for (const std::vector<int> &order : {up, down}) {
        Call c = start;
        c.a.seed = c.seed.data();
        c.a.sh = c.sh.data();
        c.a.sc = c.sc.data();
        c.a.sc_hist = c.a.sc_hist ? c.hist.data() : nullptr;
        c.a.mc = c.mc.data();
        c.a.dc = c.dc.data();
        c.a.sb = c.sb.data();
        c.a.part = c.part.data();
        std::string f = emu::run_block(nt, order.data(), [&] { kernel(c.a); });
        for (char &ch : f) if (ch == '\n') ch = ';';
        std::printf("%-44s %-5s %s run %d on %d broken %d exhausted %d\n", what, order[0] == 0 ? "up" : "down",
                    f.empty() ? "ok" : f.c_str(), c.seed[0].run, c.seed[0].bicg_on, c.seed[0].broken, c.seed[0].exhausted);
        if (!f.empty()) ++bad;
        if (order[0] == 0) first = c.seed[0];
        else if (std::memcmp(&first, &c.seed[0], sizeof(first))) {
            std::printf("%-44s the state depends on the order\n", what);
            ++bad;
        }
    }
}
}  // namespace

int main() {
    for (int then = 0; then < 2; ++then) {
        Call c(3, then);
        c.a.j = 1;
        c.a.then_basis = then;
        check(then ? "alpha, then the basis" : "alpha", SC_THREADS, c, [](ScalarArgs a) { sc_alpha(a); });
        c.row(0, 0.0);
        c.row(1, 0.0);
        check(then ? "alpha breaks down, then the basis" : "alpha breaks down", SC_THREADS, c,
              [](ScalarArgs a) { sc_alpha(a); });
    }
    for (int basis = 0; basis < 2; ++basis)
        for (int j = 0; j < 2; ++j) {
            Call c(3, basis);
            c.a.j = j;
            c.seed[0].exh_check = basis;
            check(basis ? "beta, basis form" : "beta", SC_THREADS, c, [](ScalarArgs a) { sc_beta(a); });
            Call d = c;
            d.row(3, 0.0);
            check(basis ? "beta, exhausted, basis form" : "beta, exhausted", SC_THREADS, d,
                  [](ScalarArgs a) { sc_beta(a); });
            c.row(0, 0.0);
            c.row(1, 0.0);
            check(basis ? "beta breaks down, basis form" : "beta breaks down", SC_THREADS, c,
                  [](ScalarArgs a) { sc_beta(a); });
            c.seed[0].bicg_on = 0;
            check("beta, closed", SC_THREADS, c, [](ScalarArgs a) { sc_beta(a); });
            check("exhaustion test, closed", SC_THREADS, c, [](ScalarArgs a) { sc_exh(a); });
        }
    for (double r4 : {1.0, 0.0}) {
        Call c(3, true);
        c.a.j = 2;
        c.row(4, r4);
        check(r4 > 0 ? "exhaustion test" : "exhaustion test, could fire", SC_THREADS, c, [](ScalarArgs a) { sc_exh(a); });
    }
    for (int le = 0; le <= 3; ++le) {
        Call c(3, false);
        c.seed[0].l_eff = le;
        for (int j = 0; j < le; ++j) c.seed[0].step_flag[j] = 2;
        for (int p = 0; p < 20; ++p) c.row(p, 0.01 * p);
        for (int p : {8, 14, 18}) c.row(p, 2.0);
        c.a.then_defer = 1;
        check("MR step, deferred coefficients", MR_THREADS, c, [](ScalarArgs a) { sc_mr<3>(a, BasisArgs<double>{}); });
    }
    for (int end = 0; end < 3; ++end) {
        Call c(3, false);
        c.a.then_beta = 1;
        c.seed[0].broken = end == 1;
        if (end == 2) c.row(2, 0.0);
        check("convergence, next beta", SC_THREADS, c, [](ScalarArgs a) { sc_conv(a); });
        c.seed[0].mixed = 1;
        check("reliable update", SC_THREADS, c, [](ScalarArgs a) { sc_rel(a); });
    }
    return bad != 0;
}
