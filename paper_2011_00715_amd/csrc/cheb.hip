// The Chebyshev-Jacobi smoother in FP64: its steps and spk_pc_chebyshev.
#include <cmath>

#include "chebstep.hpp"

namespace spk {
template int cheb_step<double>(spk_mat *, const ChebStep<double> &, double *, hipStream_t, int *);
}  // namespace spk

using namespace spk;

extern "C" {

int spk_pc_chebyshev(const spk_mat *Ac, const double *b, double *x, double *r_out, int32_t steps,
                     double emin, double emax, int32_t x0_nonzero, void *stream)
{
    spk_mat *A = const_cast<spk_mat *>(Ac);
    if (!A) { set_error("A is NULL"); return SPK_EINVAL; }
    const int64_t n = A->n;
    if (n > 0 && (!b || !x)) { set_error("NULL b or x"); return SPK_EINVAL; }
    if (steps < 0) { set_error("steps = %d < 0", steps); return SPK_EINVAL; }
    auto overlap = [n](const double *a, const double *c) { return a && c && a < c + n && c < a + n; };
    if (n > 0 && (overlap(b, x) || overlap(r_out, x) || overlap(r_out, b))) {
        set_error("b, x and r_out must not overlap");
        return SPK_EINVAL;
    }
    if (A->stats.zero_diag) {
        set_error("%d rows without a nonzero diagonal", A->stats.zero_diag);
        return SPK_EZERODIAG;
    }
    if (!(emax > 0.0)) emax = A->info.gershgorin;
    if (!(emin > 0.0)) emin = emax / 10.0;
    if (!(emin > 0.0) || !(emax > emin) || !std::isfinite(emax)) {
        set_error("spectral interval [%g, %g]: need 0 < emin < emax", emin, emax);
        return SPK_EINVAL;
    }
    if (n == 0) return SPK_OK;
    hipStream_t s = (hipStream_t)stream;
    A->stream = s;
    const double theta = 0.5 * (emax + emin), delta = 0.5 * (emax - emin), sigma = theta / delta;
    if (steps == 1 && !r_out && !x0_nonzero) {
        hipLaunchKernelGGL((k_cheb_one<double>), dim3(grid_n(n)), dim3(kBlock), 0, s, (int)n, b,
                           (const double *)A->dinv, 1.0 / theta, x);
        SPK_HIP(hipGetLastError());
        return SPK_OK;
    }
    // from zero on SELL the first step forms its own start
    const bool zero_fused = !x0_nonzero && steps >= 1 && cheb_zero_fused(A);
    // without a residual the last step is only x += d: the pass before adds it
    const int passes = r_out ? steps : steps - 1;
    // a single pass that starts and ends by itself keeps no vector (128^3: the
    // first call on a handle 0.55 -> 0.04 ms)
    double *r = r_out, *dbuf[2] = {nullptr, nullptr}, *tmp = nullptr;
    if (!(zero_fused && passes == 1)) {
        Workspace *w = nullptr;
        SPK_TRY(get_workspace(A, false, &w, s));
        if (!r_out) r = w->r;
        dbuf[0] = w->z;
        dbuf[1] = w->p;
        tmp = w->q;
    }
    if (!zero_fused) {
        if (x0_nonzero) SPK_TRY(launch_spmv<double>(A, A->val, x, tmp, s, nullptr, kGateNone));
        hipLaunchKernelGGL((k_cheb_init<double, double>), dim3(grid_n(n)), dim3(kBlock), 0, s, (int)n, b,
                           x0_nonzero ? (const double *)tmp : nullptr, x, r, dbuf[0], (const double *)A->dinv,
                           1.0 / theta, (const SysState *)nullptr, (double *)nullptr);
        SPK_HIP(hipGetLastError());
    }
    if (steps == 1 && !r_out) {
        hipLaunchKernelGGL((k_cheb_last<double>), dim3(grid_n(n)), dim3(kBlock), 0, s, (int)n,
                           (const double *)dbuf[0], x, (const SysState *)nullptr);
        SPK_HIP(hipGetLastError());
        return SPK_OK;
    }
    double rho = 1.0 / sigma;
    for (int k = 0; k < passes; ++k) {
        const double rho_next = 1.0 / (2.0 * sigma - rho);
        ChebStep<double> c;
        c.dk = dbuf[k & 1];
        c.dn = k == steps - 1 ? nullptr : dbuf[(k + 1) & 1];
        c.r = r;
        c.x = x;
        c.dinv = A->dinv;
        c.c1 = rho_next * rho;
        c.c2 = 2.0 * rho_next / delta;
        if (k == 0 && zero_fused) {
            c.b = b;
            c.inv_theta = 1.0 / theta;
        }
        c.close = !r_out && k == passes - 1;
        SPK_TRY(cheb_step(A, c, tmp, s));
        rho = rho_next;
    }
    return SPK_OK;
}

}  // extern "C"
