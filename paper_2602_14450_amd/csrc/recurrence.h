// The scalar recurrences of the rescaled BiCGStab (Alg. 4 / Alg. 5), advanced by
// one thread from finished sums, and the copies of a right-hand side's scalars
// that folded launches keep (ScalarFold in internal.h).
#pragma once
#include "common.h"
#include "internal.h"

namespace qcd {

__device__ __forceinline__ cx<double> cd(const double* a) { return cx<double>(a[0], a[1]); }
__device__ __forceinline__ void setc(double* a, cx<double> v) { a[0] = v.re; a[1] = v.im; }
__device__ __forceinline__ cx<double> cdiv(cx<double> a, cx<double> b) {
  const double d = b.re * b.re + b.im * b.im;
  return cx<double>((a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d);
}
__device__ __forceinline__ bool finite_c(cx<double> a) { return isfinite(a.re) && isfinite(a.im); }

// End of an inner solve; with device-driven refinement its refinement step becomes due.
__device__ inline void stop(Scalars* sc, int status) {
  sc->status = status;
  sc->active = 0;
  if (sc->dev_outer && sc->outer_active) sc->outer_step = 1;
}

// Start of a BiCGStab run: x0 = 0, r = r* = b, p = v = 0, rho' = |r|^2,
// omega' = alpha' = gamma' = lambda' = 1.
__device__ inline void bicg_init_dev(Scalars* sc, double bn2) {
  sc->bnorm2 = bn2;
  sc->rnorm2 = bn2;
  sc->rho[0] = bn2; sc->rho[1] = 0;
  sc->rho_prev[0] = bn2; sc->rho_prev[1] = 0;
  sc->alpha_prev[0] = 1; sc->alpha_prev[1] = 0;
  sc->omega_prev[0] = 1; sc->omega_prev[1] = 0;
  sc->beta[0] = 1; sc->beta[1] = 0;
  sc->pcoef[0] = 0; sc->pcoef[1] = 0;
  sc->gamma = sc->gamma_cum = sc->lambda_cum = 1.0;
  sc->xscale = 1.0;
  sc->xcoef = 1.0;
  sc->gamma_pred = 1.0;
  sc->iter = 0;
  sc->first = 1;
  sc->pending = 0;
  sc->status = kRunning;
  sc->active = 1;
  if (!(bn2 > 0.0)) stop(sc, bn2 == 0.0 ? kConverged : kNonFinite);
  else if (bn2 <= sc->tol2 * bn2) stop(sc, kConverged);
}

// alpha = rho / (r*, v)
__device__ inline void alpha_dev(Scalars* sc, const double (&s)[2]) {
  const cx<double> rv(s[0], s[1]);
  if (rv.re == 0.0 && rv.im == 0.0) { stop(sc, kBreakdown); return; }
  const cx<double> a = cdiv(cd(sc->rho), rv);
  if (!finite_c(a)) { stop(sc, kNonFinite); return; }
  setc(sc->alpha, a);
}

// omega = (t,s)/(t,t) with the omega_0 prescription; the x-update factor
// lambda'/gamma'; and the factor that rescales the new residual to norm
// sigma, from |s - omega t|^2 = (s,s) - 2 Re(conj(omega)(t,s)) + |omega|^2 (t,t).
__device__ inline void omega_dev(Scalars* sc, const double (&s)[4]) {
  const cx<double> ts(s[0], s[1]);
  const double tt = s[2], ss = s[3];
  if (!(tt > 0.0)) {  // t = A s = 0 means s = 0: the previous step solved the system
    if (ss == 0.0) {
      sc->omega[0] = 0; sc->omega[1] = 0;
    } else { stop(sc, kBreakdown); return; }
  } else {
    cx<double> om = (1.0 / tt) * ts;
    const double ah = sqrt(ts.re * ts.re + ts.im * ts.im) / sqrt(tt * ss);
    if (ah < sc->omega0) om = (sc->omega0 / ah) * om;
    setc(sc->omega, om);
  }
  const cx<double> om = cd(sc->omega);
  sc->xcoef = sc->lambda_cum / sc->gamma_cum;
  if (sc->sigma > 0.0) {
    double g2 = ss - 2.0 * (om.re * ts.re + om.im * ts.im) + (om.re * om.re + om.im * om.im) * tt;
    // below ~1e-6 (s,s) the prediction is dominated by cancellation; the
    // floor keeps the stored residual from overflowing in that case, and
    // the recalculated gamma (or the factor itself) keeps the bookkeeping exact
    const double floor2 = 1e-10 * ss;
    if (!(g2 > floor2)) g2 = floor2;
    sc->gamma_pred = (g2 > 0.0) ? sc->sigma / sqrt(g2) : 1.0;
  } else {
    sc->gamma_pred = 1.0;
  }
  if (!finite_c(om) || !isfinite(sc->gamma_pred)) stop(sc, kNonFinite);
}

// End of an iteration: gamma (applied or recalculated), rho' = gamma rho,
// gamma' *= gamma, the next rho and beta, lambda for Alg. 5, the stopping test.
// history: this right-hand side's, or null.
__device__ inline void iter_end_dev(Scalars* sc, const double (&s)[5], double* history) {
  const double ww = s[0], rr = s[1], xx = s[4];
  const cx<double> rsr(s[2], s[3]);
  double gamma = 1.0;
  if (sc->sigma > 0.0) {
    if (sc->recalc_gamma) gamma = (ww > 0.0) ? sqrt(rr / ww) : sc->gamma_pred;
    else gamma = sc->gamma_pred;
  }
  sc->gamma = gamma;
  const cx<double> rho_cur = cd(sc->rho);
  setc(sc->rho_prev, gamma * rho_cur);
  setc(sc->omega_prev, cd(sc->omega));
  setc(sc->alpha_prev, cd(sc->alpha));
  sc->gamma_cum *= gamma;
  setc(sc->rho, rsr);
  // beta for the next iteration and the folded p/v rescaling
  const cx<double> beta = cdiv(rsr * cd(sc->alpha_prev), cd(sc->rho_prev) * cd(sc->omega_prev));
  setc(sc->beta, beta);
  setc(sc->pcoef, gamma * beta);
  // Alg. 5: lambda = sigma_lambda / |x|, applied to x at the next update
  if (sc->sigma_lambda > 0.0 && xx > 0.0) {
    const double lam = sc->sigma_lambda / sqrt(xx);
    sc->xscale = lam;
    sc->lambda_cum *= lam;
  } else {
    sc->xscale = 1.0;
  }
  sc->rnorm2 = rr;
  sc->first = 0;
  const double res2 = rr / (sc->gamma_cum * sc->gamma_cum);
  if (history && sc->iter < sc->max_iter) history[sc->iter] = res2;
  sc->iter += 1;
  if (!isfinite(res2) || !finite_c(beta) || !isfinite(sc->lambda_cum) || !isfinite(sc->gamma_cum)) {
    // an exact zero residual ends the run as converged
    if (rr == 0.0 && ww == 0.0) stop(sc, kConverged);
    else stop(sc, kNonFinite);
    return;
  }
  if (res2 <= sc->tol2 * sc->bnorm2) { stop(sc, kConverged); return; }
  if (rsr.re == 0.0 && rsr.im == 0.0) { stop(sc, kBreakdown); return; }
  if (sc->iter >= sc->max_iter) stop(sc, kMaxIter);
}

// Scalars inside the vector kernels (ScalarFold).  alpha, omega and the end of
// an iteration each need a sum over the partial rows of the launch before.  On
// a small lattice a launch of its own for that costs as much as any other (the
// host enqueues one in 3-4 us, and the GPU takes 4-5 us for it), so every block
// of the launch that needs the scalar sums the rows itself (in the same order,
// so all blocks get the same bits) while its first vector loads are in flight,
// and block 0 records the result.  No block may read what block 0 writes, so
// the scalars live in three copies, and each launch that advances them reads one
// and writes another: the one that takes the direction update reads `sc`,
// applies the pending end of the last iteration and writes `next`; the one that
// takes s = r - alpha v reads `next` and writes `mid` with alpha; the x / r
// update reads `mid` and writes `sc` back with omega and the pending mark.
__device__ __forceinline__ void copy_scalars(Scalars* dst, const Scalars* src) {
  constexpr int words = sizeof(Scalars) / sizeof(uint32_t);
  for (int i = threadIdx.x; i < words; i += blockDim.x)
    reinterpret_cast<uint32_t*>(dst)[i] = reinterpret_cast<const uint32_t*>(src)[i];
}
// This block's copy sh of the scalars with the pending end of the last
// iteration applied, and block 0's record of it in next[rhs].
__device__ __forceinline__ void fold_iter_end(Scalars& sh, const Scalars* sc, Scalars* next, const double* rows,
                                              int nrows, double* history, int hist_stride, int rhs) {
  copy_scalars(&sh, sc + rhs);
  double s[5];
  finish_sum<5>(rows + (size_t)rhs * nrows * 5, nrows, s);
  if (threadIdx.x == 0 && sh.active && sh.pending) {
    sh.pending = 0;
    iter_end_dev(&sh, s, history && blockIdx.x == 0 ? history + (size_t)rhs * hist_stride : nullptr);
  }
  __syncthreads();
  if (blockIdx.x == 0) copy_scalars(next + rhs, &sh);
}
// The same with alpha, recorded in mid[rhs].
__device__ __forceinline__ void fold_alpha(Scalars& sh, const Scalars* next, Scalars* mid, const double* rows,
                                           int nrows, int rhs) {
  copy_scalars(&sh, next + rhs);
  double s[2];
  finish_sum<2>(rows + (size_t)rhs * nrows * 2, nrows, s);
  if (threadIdx.x == 0 && sh.active) alpha_dev(&sh, s);
  __syncthreads();
  if (blockIdx.x == 0) copy_scalars(mid + rhs, &sh);
}
// The same with omega and the pending mark, recorded in sc[rhs].
__device__ __forceinline__ void fold_omega(Scalars& sh, const Scalars* mid, Scalars* sc, const double* rows, int nrows,
                                           int rhs) {
  copy_scalars(&sh, mid + rhs);
  double s[4];
  finish_sum<4>(rows + (size_t)rhs * nrows * 4, nrows, s);
  if (threadIdx.x == 0 && sh.active) {
    omega_dev(&sh, s);
    sh.pending = sh.active;
  }
  __syncthreads();
  if (blockIdx.x == 0) copy_scalars(sc + rhs, &sh);
}

}  // namespace qcd
