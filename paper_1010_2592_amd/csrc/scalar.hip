// Device-side scalar work of multi-shift BiCGstab(l): one block per
// right-hand side, FP64 throughout.  Keeping these steps on the device means
// the host never waits on an inner product inside an outer iteration: the
// vector kernels read the coefficients these kernels write, and a right-hand
// side that has stopped (or whose BiCG part has ended early) gates every later
// launch off through its SeedState flags.
//
// Seed (BiCGstab(l), x0 = 0, shadow residual b):
//   j = 0: rho0 <- -omega rho0
//   rho1 = <rt, r_j>, beta = alpha rho1 / rho0, rho0 = rho1
//   gamma = <rt, u_{j+1}>, alpha = rho0 / gamma
//   MR: G g = c by Cholesky, G_ik = <r_i, r_k>, c_i = <r_i, r_0>, omega = g_l
// Shifts (sigma' = sigma_s - sigma_0; zeta_n = R_n(-sigma'), pi_n = P_n(-sigma'),
// psi = product of the MR polynomials at -sigma'):
//   pi_n = zeta_n - beta_n pi_{n-1},  zeta_{n+1} = zeta_n + alpha_n sigma' pi_n
//   alpha^s = alpha zeta_n / zeta_{n+1},  beta^s = beta (zeta_{n-1} / zeta_n)^2
//   kappa_n = 1 / (zeta_n psi)
//   MR: q^s = 1 - sum_i g_i (-sigma')^i,
//       c^s_k = (1/q^s) sum_{i>k} g_i (-sigma')^{i-1-k},  psi <- psi q^s
// Convergence at the end of each outer iteration: shift s freezes when
// ||r_0|| / (|zeta psi| ||b||) <= tol (its outer-iteration count is the
// paper's M_s, Section 2); the iteration stops when no shift is left.
#include "scalar_dev.h"

namespace msb {

namespace {

using namespace dev;

__global__ __launch_bounds__(BLOCK) void sc_init(ScalarArgs a) { sc_init_body(a, blockIdx.x); }
__global__ __launch_bounds__(SC_THREADS) void sc_beta(ScalarArgs a) {
    __shared__ StateLds l;
    StageState<SC_THREADS> st(a, blockIdx.x, l);
    sc_beta_body(a, blockIdx.x, st);
    st.leave();
}
__global__ __launch_bounds__(SC_THREADS) void sc_alpha(ScalarArgs a) {
    __shared__ StateLds l;
    StageState<SC_THREADS> st(a, blockIdx.x, l);
    sc_alpha_body(a, blockIdx.x, st);
    if (a.then_basis) {
        __syncthreads();   // the steps' flags and coefficients, written by one work-item
        sc_basis_body(a, blockIdx.x, st.S);
    }
    st.leave();
}
// The MR stage and what follows from its coefficients alone (512 work-items:
// the deferred coefficients keep three columns of L + 1 in registers)
constexpr int MR_THREADS = 512;
template <int L>
__global__ __launch_bounds__(MR_THREADS) void sc_mr(ScalarArgs a, BasisArgs<double> b) {
    __shared__ StateLds l;
    StageState<MR_THREADS> st(a, blockIdx.x, l);
    sc_mr_body<L>(a, blockIdx.x, st);
    __syncthreads();
    if (b.sp_cnt) basis_spec_body<L>(b, blockIdx.x, st.S);
    if (a.then_defer) sc_defer_body<L>(a, blockIdx.x, st.S);
    st.leave();
}
__global__ __launch_bounds__(SC_THREADS) void sc_rel(ScalarArgs a) {
    __shared__ StateLds l;
    StageState<SC_THREADS> st(a, blockIdx.x, l);
    sc_rel_body(a, blockIdx.x, st);
    st.leave();
}
__global__ __launch_bounds__(SC_THREADS) void sc_conv(ScalarArgs a) {
    __shared__ StateLds l;
    StageState<SC_THREADS> st(a, blockIdx.x, l);
    sc_conv_body(a, blockIdx.x, st);
    st.leave();
}
__global__ __launch_bounds__(SC_THREADS) void sc_exh(ScalarArgs a) {
    __shared__ StateLds l;
    StageState<SC_THREADS> st(a, blockIdx.x, l);
    sc_exh_body(a, blockIdx.x, st);
    st.leave();
}
__global__ __launch_bounds__(64) void sc_basis_replay(BasisReplayArgs a) { sc_basis_replay_body(a, blockIdx.x); }

}  // namespace

void launch_sc_init(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_init, dim3(nrhs), dim3(BLOCK), 0, st, a);
}
void launch_sc_beta(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_beta, dim3(nrhs), dim3(SC_THREADS), 0, st, a);
}
void launch_sc_alpha(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_alpha, dim3(nrhs), dim3(SC_THREADS), 0, st, a);
}
void launch_sc_mr(hipStream_t st, const ScalarArgs &a, const BasisArgs<double> *spec, int nrhs) {
    const BasisArgs<double> b = spec ? *spec : BasisArgs<double>{};
    switch (a.l) {
#define C_(L) case L: hipLaunchKernelGGL((sc_mr<L>), dim3(nrhs), dim3(MR_THREADS), 0, st, a, b); break;
        C_(1) C_(2) C_(3) C_(4) C_(5) C_(6) C_(7) C_(8)
#undef C_
    }
}
void launch_sc_rel(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_rel, dim3(nrhs), dim3(SC_THREADS), 0, st, a);
}
void launch_sc_conv(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_conv, dim3(nrhs), dim3(SC_THREADS), 0, st, a);
}
void launch_sc_exh(hipStream_t st, const ScalarArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_exh, dim3(nrhs), dim3(SC_THREADS), 0, st, a);
}
void launch_sc_basis_replay(hipStream_t st, const BasisReplayArgs &a, int nrhs) {
    hipLaunchKernelGGL(sc_basis_replay, dim3(nrhs), dim3(64), 0, st, a);
}

}  // namespace msb
