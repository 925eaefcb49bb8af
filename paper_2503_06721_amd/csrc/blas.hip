// Linear algebra on packed half spinors and the per-iteration kernels of the
// conjugate-gradient solver.  Sums are accumulated in FP64 whatever the field
// precision; block partial sums are combined by one block per right-hand
// side with Neumaier's compensated summation (Sec. 5.1.1), in a fixed order,
// so results are deterministic (no floating-point atomics).
#include "wd_common.h"
#include "wd_kernels.h"

namespace wd {

constexpr int BT = 256;   // threads per block of the streaming kernels

int blas_nblocks(const FieldShape &f) { return (f.maxvh + BT - 1) / BT; }

Counts uniform_counts(int n) {
  Counts c;
  for (int k = 0; k < MAXSYS; ++k) c.n[k] = n;
  return c;
}

// Row addressing of system s: element (component c, site i) is at
// f.off[s] + c * f.stride[s] + i.

template <typename T>
__device__ __forceinline__ cplx<T> ld(const void *p, size_t o) {
  return static_cast<const cplx<T> *>(p)[o];
}
template <typename T>
__device__ __forceinline__ void st(void *p, size_t o, cplx<double> v) {
  static_cast<cplx<T> *>(p)[o] = mk<T>((T)v.re, (T)v.im);
}
template <typename T>
__device__ __forceinline__ cplx<double> up(cplx<T> v) {
  return mk<double>((double)v.re, (double)v.im);
}

__global__ __launch_bounds__(BT) void k_finalize_sum(double *out, const double *partial, int prow, Counts cnt,
                                                     int nsys) {
  const int r = blockIdx.x;
  const double s = sum_partials(partial + (size_t)r * prow, cnt.n[r % nsys]);
  if (threadIdx.x == 0) out[r] = s;
}

// One block per row; rows r >= nsys (the imaginary parts of dot products)
// use the counts of system r - nsys.
hipError_t launch_finalize_sum(double *out, const double *partial, int prow, const Counts &counts, int nrows,
                               int nsys, hipStream_t st) {
  hipLaunchKernelGGL(k_finalize_sum, dim3(nrows), dim3(BT), 0, st, out, partial, prow, counts, nsys);
  return hipGetLastError();
}

// ------------------------------------------------------------- streaming
template <typename T>
__global__ __launch_bounds__(BT) void k_lincomb(void *out, double a, const void *x, double b, const void *y,
                                                FieldShape f) {
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  if (i >= f.vh[sy]) return;
  const size_t base = (size_t)f.off[sy] + i;
  for (int c = 0; c < f.ncomp; ++c) {
    const size_t o = base + (size_t)c * f.stride[sy];
    cplx<double> v = up(ld<T>(x, o));
    v = a * v;
    if (y) {
      const cplx<double> w = up(ld<T>(y, o));
      v.re = fma(b, w.re, v.re);
      v.im = fma(b, w.im, v.im);
    }
    st<T>(out, o, v);
  }
}

hipError_t launch_lincomb(void *out, double a, const void *x, double b, const void *y, const FieldShape &f, int prec,
                          hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  if (prec == 0) hipLaunchKernelGGL(k_lincomb<double>, grid, dim3(BT), 0, st, out, a, x, b, y, f);
  else hipLaunchKernelGGL(k_lincomb<float>, grid, dim3(BT), 0, st, out, a, x, b, y, f);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(BT) void k_norm2_partial(double *partial, const void *v, FieldShape f) {
  __shared__ double sh[BT / 64];
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  double s = 0.0;
  if (i < f.vh[sy]) {
    const size_t base = (size_t)f.off[sy] + i;
    for (int c = 0; c < f.ncomp; ++c) {
      const cplx<T> w = ld<T>(v, base + (size_t)c * f.stride[sy]);
      s += (double)w.re * w.re + (double)w.im * w.im;
    }
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

hipError_t launch_norm2_partial(double *partial, const void *v, const FieldShape &f, int prec, hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  if (prec == 0) hipLaunchKernelGGL(k_norm2_partial<double>, grid, dim3(BT), 0, st, partial, v, f);
  else hipLaunchKernelGGL(k_norm2_partial<float>, grid, dim3(BT), 0, st, partial, v, f);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(BT) void k_dot_partial(double *partial, const void *a, const void *b, FieldShape f) {
  __shared__ double sh[BT / 64];
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  double re = 0.0, im = 0.0;
  if (i < f.vh[sy]) {
    const size_t base = (size_t)f.off[sy] + i;
    for (int c = 0; c < f.ncomp; ++c) {
      const size_t o = base + (size_t)c * f.stride[sy];
      const cplx<double> x = up(ld<T>(a, o)), y = up(ld<T>(b, o));
      re = fma(x.re, y.re, re);
      re = fma(x.im, y.im, re);
      im = fma(x.re, y.im, im);
      im = fma(-x.im, y.re, im);
    }
  }
  re = block_sum(re, sh);
  im = block_sum(im, sh);
  if (threadIdx.x == 0) {
    partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = re;
    partial[(size_t)(gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = im;
  }
}

hipError_t launch_dot_partial(double *partial, const void *a, const void *b, const FieldShape &f, int prec,
                              hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  if (prec == 0) hipLaunchKernelGGL(k_dot_partial<double>, grid, dim3(BT), 0, st, partial, a, b, f);
  else hipLaunchKernelGGL(k_dot_partial<float>, grid, dim3(BT), 0, st, partial, a, b, f);
  return hipGetLastError();
}

template <typename TO, typename TI>
__global__ __launch_bounds__(BT) void k_convert(void *out, const void *in, FieldShape f) {
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  if (i >= f.vh[sy]) return;
  const size_t base = (size_t)f.off[sy] + i;
  for (int c = 0; c < f.ncomp; ++c) {
    const size_t o = base + (size_t)c * f.stride[sy];
    st<TO>(out, o, up(ld<TI>(in, o)));
  }
}

hipError_t launch_convert(void *out, int prec_out, const void *in, int prec_in, const FieldShape &f,
                          hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  if (prec_out == 0 && prec_in == 1) hipLaunchKernelGGL((k_convert<double, float>), grid, dim3(BT), 0, st, out, in, f);
  else if (prec_out == 1 && prec_in == 0) hipLaunchKernelGGL((k_convert<float, double>), grid, dim3(BT), 0, st, out, in, f);
  else if (prec_out == 0) hipLaunchKernelGGL((k_convert<double, double>), grid, dim3(BT), 0, st, out, in, f);
  else hipLaunchKernelGGL((k_convert<float, float>), grid, dim3(BT), 0, st, out, in, f);
  return hipGetLastError();
}

// ------------------------------------------------------------------- CG
// State of a system at the end of an iteration, rr = |r|^2 after it (thread 0
// of one block).
__device__ __forceinline__ void cg_end_step(CgScalars &s, double rr, double delta) {
  s.iters += 1;
  if (!isfinite(rr)) {
    s.status = -5;
    s.active = 0;
    return;
  }
  s.rho = rr;
  const double rn = sqrt(rr);
  if (rn > s.rmax) s.rmax = rn;
  if (rr <= s.stop2) {
    s.active = 0;          // recursive residual converged: verify in FP64
    s.need_update = 1;
  } else if (delta > 0.0 && rn < delta * s.rmax) {
    // mixed mode: ask for a reliable update and keep iterating until every
    // other active system asks too, so that no system idles while the
    // batched hops still stream its field
    s.need_update = 1;
  }
}

// The sum and the state update as a kernel of their own, one block per system.
__global__ __launch_bounds__(1024) void k_cg_end(CgScalars *S, const double *__restrict__ rr_partial, int prow,
                                                 Counts cnt, double delta) {
  CgScalars &s = S[blockIdx.x];
  if (!s.act_it) return;
  const double rr = sum_partials(rr_partial + (size_t)blockIdx.x * prow, cnt.n[blockIdx.x]);
  if (threadIdx.x != 0) return;
  s.rr = rr;
  cg_end_step(s, rr, delta);
}

// End of an iteration: beta = rho'/rho from the partial sums of |r|^2 that the
// last hop left, x += alpha p, p = r + beta p, and the state of the system
// (convergence, and in mixed mode the reliable-update trigger).
//
// Bound by memory: x, p read and written, r read (5 half fields; with r's own
// update in the hop an iteration moves 6 beside its hops instead of 9 and a
// stored A p): 6.4 TB/s on SU(3) FUND 32^4 (FP32 40 us, where the separate
// x, r and p updates took 72).  Up to kOwnSum partial sums every block adds
// them up itself (OWN), which costs less than a launch between the hop and
// this kernel; the first block of a system then stores the state, whose
// fields no block reads here.  Longer rows are summed by k_cg_end (2592
// partial sums, SU(3) FUND 24^4: 32.1 us with them, 27.6 + 5.5 us and a launch
// apart; 8192, 32^4 FP32: 47.1 against 40.9 + 5.5 us).
// Thread per site and, by blockIdx.z, group of `per` components: all 4 d of
// them where the sites alone give every CU four blocks, else four, which
// shortens the chain of loads of a small lattice (SU(2) ADJ 32x16^3: 13.0 us,
// the separate updates 23.6; SU(2) FUND 4^4: 3.5, they 7.9).
constexpr int kOwnSum = 4096;
template <typename T, bool OWN>
__global__ __launch_bounds__(BT) void k_cg_update_xp(cplx<T> *__restrict__ x, cplx<T> *__restrict__ p,
                                                     const cplx<T> *__restrict__ r, CgScalars *S,
                                                     const double *__restrict__ rr_partial, int prow, Counts cnt,
                                                     double delta, int per, FieldShape f) {
  const int sy = blockIdx.y;
  CgScalars &s = S[sy];
  const int i = blockIdx.x * BT + threadIdx.x;
  const bool in = i < f.vh[sy];
  const size_t st = f.stride[sy];
  const size_t base = (size_t)f.off[sy] + i + (size_t)blockIdx.z * per * st;
  cplx<T> pv[4], xv[4], rv[4];
  const auto load = [&](int c) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t o = base + (size_t)(c + k) * st;
      pv[k] = p[o];
      xv[k] = x[o];
      rv[k] = r[o];
    }
  };
  if (in) load(0);   // on their way while the partial sums are added up
  if (!s.act_it) return;
  const double a = s.alpha, rho = s.rho_it;
  double rr;
  if constexpr (OWN) {
    rr = sum_partials(rr_partial + (size_t)sy * prow, cnt.n[sy]);
    if (blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) cg_end_step(s, rr, delta);
  } else {
    rr = s.rr;
  }
  if (!in) return;
  const bool ok = isfinite(rr);
  const double b = rr / rho;
  for (int c = 0;;) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t o = base + (size_t)(c + k) * st;
      x[o] = mk<T>((T)fma(a, (double)pv[k].re, (double)xv[k].re), (T)fma(a, (double)pv[k].im, (double)xv[k].im));
      // a residual that is not finite ends the system before its p update
      if (ok)
        p[o] = mk<T>((T)fma(b, (double)pv[k].re, (double)rv[k].re), (T)fma(b, (double)pv[k].im, (double)rv[k].im));
    }
    c += 4;
    if (c >= per) return;
    load(c);
  }
}

template <typename T>
static void update_xp(void *x, void *p, const void *r, CgScalars *s, const double *rr_partial, int prow,
                      const Counts &counts, double delta, const FieldShape &f, hipStream_t st) {
  const int nb = blas_nblocks(f);
  const int per = nb * f.nsys >= 1024 ? f.ncomp : 4;
  const dim3 grid(nb, f.nsys, f.ncomp / per);
  if (prow <= kOwnSum) {
    hipLaunchKernelGGL((k_cg_update_xp<T, true>), grid, dim3(BT), 0, st, (cplx<T> *)x, (cplx<T> *)p,
                       (const cplx<T> *)r, s, rr_partial, prow, counts, delta, per, f);
  } else {
    hipLaunchKernelGGL(k_cg_end, dim3(f.nsys), dim3(1024), 0, st, s, rr_partial, prow, counts, delta);
    hipLaunchKernelGGL((k_cg_update_xp<T, false>), grid, dim3(BT), 0, st, (cplx<T> *)x, (cplx<T> *)p,
                       (const cplx<T> *)r, s, rr_partial, prow, counts, delta, per, f);
  }
}

hipError_t launch_cg_update_xp(void *x, void *p, const void *r, CgScalars *s, const double *rr_partial, int prow,
                               const Counts &counts, double delta, const FieldShape &f, int prec, hipStream_t st) {
  if (prec == 0) update_xp<double>(x, p, r, s, rr_partial, prow, counts, delta, f, st);
  else update_xp<float>(x, p, r, s, rr_partial, prow, counts, delta, f, st);
  return hipGetLastError();
}

// After a (re)computation of r = b - A x in FP64: rho = ||r||^2.  With set_b2
// the partial sums are those of b itself and only b2 / stop2 are set.
// Otherwise rhs that are not finished are (re)activated: finished means
// converged (rho <= stop2), broken down, or b = 0. 
__global__ __launch_bounds__(BT) void k_cg_restart(CgScalars *S, const double *partial, int prow, Counts cnt,
                                                   double tol, int set_b2) {
  const int r = blockIdx.x;
  CgScalars &s = S[r];
  const double v = sum_partials(partial + (size_t)r * prow, cnt.n[r]);
  if (threadIdx.x != 0) return;
  if (set_b2) {
    s.b2 = v;
    s.stop2 = tol * tol * v;
    s.iters = 0;
    s.status = 0;
    s.active = s.act_it = 0;
    s.need_update = 0;
    s.rmax = 0.0;
    return;
  }
  s.rho = v;
  s.rmax = sqrt(v);
  s.need_update = 0;
  if (s.status != 0) {
    s.active = 0;
    return;
  }
  if (!isfinite(v)) {
    s.status = -5;
    s.active = 0;
    return;
  }
  s.active = (s.b2 > 0.0 && v > s.stop2) ? 1 : 0;
}

hipError_t launch_cg_restart(CgScalars *s, const double *partial, int prow, const Counts &counts, int nsys, double tol,
                             int set_b2, hipStream_t st) {
  hipLaunchKernelGGL(k_cg_restart, dim3(nsys), dim3(BT), 0, st, s, partial, prow, counts, tol, set_b2);
  return hipGetLastError();
}

// x64 += x32 and x32 = 0 (mixed-mode accumulation of the inner solution).
__global__ __launch_bounds__(BT) void k_accum_x(void *x64, void *x32, FieldShape f) {
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  if (i >= f.vh[sy]) return;
  const size_t base = (size_t)f.off[sy] + i;
  for (int c = 0; c < f.ncomp; ++c) {
    const size_t o = base + (size_t)c * f.stride[sy];
    const cplx<double> v = ld<double>(x64, o) + up(ld<float>(x32, o));
    st<double>(x64, o, v);
    st<float>(x32, o, mk(0.0, 0.0));
  }
}

hipError_t launch_accum_x(void *x64, void *x32, const FieldShape &f, hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  hipLaunchKernelGGL(k_accum_x, grid, dim3(BT), 0, st, x64, x32, f);
  return hipGetLastError();
}

// out = gamma_5 x + i c y (y nullable), gamma_5 = diag(1, 1, -1, -1) on the
// spin index (components spin * d + colour); out may alias x or y.
template <typename T>
__global__ __launch_bounds__(BT) void k_gamma5_axpy(void *out, const void *x, double c, const void *y,
                                                    FieldShape f) {
  const int i = blockIdx.x * BT + threadIdx.x, sy = blockIdx.y;
  if (i >= f.vh[sy]) return;
  const size_t base = (size_t)f.off[sy] + i;
  const int d = f.ncomp / 4;
  for (int comp = 0; comp < f.ncomp; ++comp) {
    const size_t o = base + (size_t)comp * f.stride[sy];
    cplx<double> v = up(ld<T>(x, o));
    if (comp >= 2 * d) v = mk(-v.re, -v.im);
    if (y) {
      const cplx<double> w = up(ld<T>(y, o));
      v.re = fma(-c, w.im, v.re);
      v.im = fma(c, w.re, v.im);
    }
    st<T>(out, o, v);
  }
}

hipError_t launch_gamma5_axpy(void *out, const void *x, double c, const void *y, const FieldShape &f, int prec,
                              hipStream_t st) {
  dim3 grid(blas_nblocks(f), f.nsys);
  if (prec == 0) hipLaunchKernelGGL(k_gamma5_axpy<double>, grid, dim3(BT), 0, st, out, x, c, y, f);
  else hipLaunchKernelGGL(k_gamma5_axpy<float>, grid, dim3(BT), 0, st, out, x, c, y, f);
  return hipGetLastError();
}

// ------------------------------------------------------------ multi-shift CG
// Recursion of the base system (smallest shift sigma0) plus, for every shift
// k with delta_k = sigma_k - sigma0 >= 0, the collinear shifted residual
// r_k = zeta_k r.  With a_{-1} = 1, b_{-1} = 0, zeta_{-1} = zeta_0 = 1:
//   zeta_k' = zeta_k zeta_k^old a_old / (a b_old (zeta_k^old - zeta_k)
//                                        + zeta_k^old a_old (1 + delta_k a)),
//   alpha_k = a zeta_k' / zeta_k,   beta_k = b (zeta_k' / zeta_k)^2,
//   x_k += alpha_k p_k,   p_k = zeta_k' r' + beta_k p_k.
// The base shift has delta = 0 and zeta = 1 throughout.  Only its p feeds the
// operator, so the updates of the other shifts wait until MSRING iterations
// can be applied in one pass over x_k and p_k (launch_ms_update_xp), from the
// residuals kept in a ring and the scalars kept per ring slot.
__global__ void k_ms_init(MsScalars *S, const double *b2_partial, int nblk, ShiftList d, int nshift, int base,
                          double sigma0, double tol) {
  const double b2 = sum_partials(b2_partial, nblk);
  if (threadIdx.x != 0) return;
  MsScalars &s = *S;
  s.cg.b2 = b2;
  s.cg.stop2 = tol * tol * b2;
  s.cg.rho = b2;
  s.cg.pAp = 0.0;
  s.cg.alpha = 0.0;
  s.cg.act_it = s.cg.need_update = 0;
  s.cg.iters = 0;
  s.alpha_old = 1.0;
  s.beta_old = 0.0;
  s.sigma0 = sigma0;
  s.nshift = nshift;
  s.base = base;
  s.xb_it = 0;
  // a non-finite right-hand side is a breakdown, not a zero source
  s.cg.status = isfinite(b2) ? 0 : -5;
  s.cg.active = (b2 > 0.0 && isfinite(b2)) ? 1 : 0;
  for (int k = 0; k < MAXSHIFT; ++k) {
    s.delta[k] = k < nshift ? d.v[k] : 0.0;
    s.zeta[k] = s.zeta_old[k] = s.zeta_new[k] = 1.0;
    s.sact[k] = k < nshift ? s.cg.active : 0;
    s.siters[k] = 0;
  }
}

hipError_t launch_ms_init(MsScalars *s, const double *b2_partial, int nblk, const ShiftList &delta, int nshift,
                          int base, double sigma0, double tol, hipStream_t st) {
  hipLaunchKernelGGL(k_ms_init, dim3(1), dim3(BT), 0, st, s, b2_partial, nblk, delta, nshift, base, sigma0, tol);
  return hipGetLastError();
}

// Scalars of every shift at the end of an iteration (one block, a thread per
// shift): beta_k, rotation of the zeta history, convergence of each shift
// (|zeta_k| ||r|| <= tol ||b||: its update of this iteration is its last), and
// the ring slot's coefficients.  The base recursion runs while any shift is
// still being updated.
__device__ __forceinline__ void ms_end_step(MsScalars &s, double rr, int slot) {
  const int k = threadIdx.x;
  const int act = s.cg.act_it;
  const bool ok = act && isfinite(rr);
  const double b = rr / s.cg.rho_it, stop2 = s.cg.stop2;
  __shared__ int any;
  if (k == 0) any = 0;
  __syncthreads();
  if (k < s.nshift) {
    const int on = s.sact[k];
    int upd = 0;
    if (ok && on) {
      const double z = s.zeta[k], zn = s.zeta_new[k], q = zn / z;
      s.as[slot][k] = s.cg.alpha * zn / z;
      s.bs[slot][k] = b * q * q;
      s.zr[slot][k] = zn;
      s.zeta_old[k] = z;
      s.zeta[k] = zn;
      s.siters[k] += 1;
      const bool more = zn * zn * rr > stop2;
      if (!more) s.sact[k] = 0;
      else any = 1;
      upd = more ? 3 : 1;
    } else if (act && !ok) {
      s.sact[k] = 0;
    }
    s.upd[slot][k] = upd;
  }
  __syncthreads();
  if (k != 0 || !act) return;
  s.cg.iters += 1;
  if (!ok) {
    s.cg.status = -5;
    s.cg.active = 0;
    return;
  }
  s.alpha_old = s.cg.alpha;
  s.beta_old = b;
  s.cg.rho = rr;
  s.cg.active = any;
}

// The sum and ms_end_step as a kernel of their own.
__global__ __launch_bounds__(1024) void k_ms_end(MsScalars *S, const double *__restrict__ rr_partial, int cnt,
                                                 int slot) {
  MsScalars &s = *S;
  const int act = s.cg.act_it;
  const double rr = act ? sum_partials(rr_partial, cnt) : 0.0;
  ms_end_step(s, rr, slot);
  if (threadIdx.x == 0) s.cg.rr = rr;
}

// Base shift: x += alpha p, p = r + beta p as k_cg_update_xp, and |p|^2 summed on
// the way where the next step length needs it (sigma0 > 0), which saves a pass
// over p.  Up to kOwnSum partial sums every block adds them up itself (OWN) and
// the first one also advances the scalars of every shift, whose fields no other
// block reads; longer rows, whose reads by every block would grow as the square
// of the volume, are summed by k_ms_end (an iteration of a one-shift solve, every
// block adding against k_ms_end: SU(3) FUND 32^4, 8192 partial sums, 739 and 734
// us; SU(2) FUND 64^4, 131072, 9.55 and 8.16 ms).
template <bool OWN>
__global__ __launch_bounds__(BT) void k_ms_update_base(cplx<double> *__restrict__ x, cplx<double> *__restrict__ p,
                                                       const cplx<double> *__restrict__ r, MsScalars *S,
                                                       const double *__restrict__ rr_partial, int cnt, int slot,
                                                       double *__restrict__ pp, int per, FieldShape f) {
  __shared__ double sh[BT / 64];
  MsScalars &s = *S;
  const int act = s.cg.act_it, xb = s.xb_it;
  const double a = s.cg.alpha, rho = s.cg.rho_it;
  double rr = 0.0;
  if constexpr (OWN) {
    if (act) rr = sum_partials(rr_partial, cnt);
    if (blockIdx.x == 0 && blockIdx.y == 0) ms_end_step(s, rr, slot);
  } else {
    rr = s.cg.rr;
  }
  if (!act) return;
  const bool ok = isfinite(rr);
  const double b = rr / rho;
  const int i = blockIdx.x * BT + threadIdx.x;
  double n = 0.0;
  if (ok && i < f.vh[0]) {
    const size_t st = f.stride[0];
    const size_t base = (size_t)f.off[0] + i + (size_t)blockIdx.y * per * st;
    for (int c = 0; c < per; c += 4) {
      cplx<double> pv[4], xv[4], rv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const size_t o = base + (size_t)(c + k) * st;
        pv[k] = p[o];
        xv[k] = x[o];
        rv[k] = r[o];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const size_t o = base + (size_t)(c + k) * st;
        if (xb) x[o] = mk(fma(a, pv[k].re, xv[k].re), fma(a, pv[k].im, xv[k].im));
        const cplx<double> pn = mk(fma(b, pv[k].re, rv[k].re), fma(b, pv[k].im, rv[k].im));
        p[o] = pn;
        n += pn.re * pn.re + pn.im * pn.im;
      }
    }
  }
  if (pp) {
    n = block_sum(n, sh);
    if (threadIdx.x == 0) pp[blockIdx.y * gridDim.x + blockIdx.x] = n;
  }
}

// Components per thread of the base update (as update_xp), and its blocks, each
// with a partial sum of |p|^2.
static int ms_base_per(const FieldShape &f) { return blas_nblocks(f) >= 1024 ? f.ncomp : 4; }
int ms_base_blocks(const FieldShape &f) { return blas_nblocks(f) * (f.ncomp / ms_base_per(f)); }

hipError_t launch_ms_update_base(void *x, void *p, const void *r, MsScalars *s, const double *rr_partial, int cnt,
                                 int slot, double *pp, const FieldShape &f, hipStream_t st) {
  const int per = ms_base_per(f);
  const dim3 grid(blas_nblocks(f), f.ncomp / per);
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(BT), 0, st, (cplx<double> *)x, (cplx<double> *)p, (const cplx<double> *)r, s,
                       rr_partial, cnt, slot, pp, per, f);
    return hipGetLastError();
  };
  if (cnt <= kOwnSum) return go(k_ms_update_base<true>);
  hipLaunchKernelGGL(k_ms_end, dim3(1), dim3(1024), 0, st, s, rr_partial, cnt, slot);
  return go(k_ms_update_base<false>);
}

// The other shifts, N iterations at once: for every slot j in turn
// x_k += as_jk p_k and p_k = zr_jk r_j + bs_jk p_k, where due.  Bound by memory:
// 4 half fields per shift and N residuals, against 4 N per shift when every
// iteration updates them (SU(3) FUND 32x24^3, 12 shifts: 342 us an iteration
// before, 368 us in eight iterations now).  One thread per site with the
// shifts in an inner loop, so that each residual is read once for all of them.
template <int N>
__global__ __launch_bounds__(BT) void k_ms_update_xp(cplx<double> *__restrict__ x, cplx<double> *__restrict__ p,
                                                     const cplx<double> *__restrict__ ring,
                                                     const MsScalars *__restrict__ S, long long fstride,
                                                     FieldShape f) {
  const MsScalars &s = *S;
  const int i = blockIdx.x * BT + threadIdx.x;
  if (i >= f.vh[0]) return;
  const int ns = s.nshift, kb = s.base;
  const size_t o = (size_t)f.off[0] + i + (size_t)blockIdx.y * f.stride[0];
  cplx<double> r[N];
#pragma unroll
  for (int j = 0; j < N; ++j) r[j] = ring[(size_t)j * fstride + o];
  for (int k = 0; k < ns; ++k) {
    if (k == kb || !s.upd[0][k]) continue;   // uniform over the grid; once off, off in the later slots
    const size_t ok = (size_t)k * fstride + o;
    cplx<double> pv = p[ok], xv = x[ok];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int u = s.upd[j][k];
      if (u & 1) {
        const double a = s.as[j][k];
        xv.re = fma(a, pv.re, xv.re);
        xv.im = fma(a, pv.im, xv.im);
      }
      if (u & 2) {
        const double z = s.zr[j][k], b = s.bs[j][k];
        pv.re = fma(z, r[j].re, b * pv.re);
        pv.im = fma(z, r[j].im, b * pv.im);
      }
    }
    x[ok] = xv;
    p[ok] = pv;
  }
}

hipError_t launch_ms_update_xp(void *x, void *p, const void *ring, const MsScalars *s, long long fstride,
                               const FieldShape &f, int n, hipStream_t st) {
  const dim3 grid(blas_nblocks(f), f.ncomp);
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(BT), 0, st, (cplx<double> *)x, (cplx<double> *)p, (const cplx<double> *)ring,
                       s, fstride, f);
    return hipGetLastError();
  };
  static_assert(MSRING == 8, "one instance per number of iterations");
  switch (n) {
    case 1: return go(k_ms_update_xp<1>);
    case 2: return go(k_ms_update_xp<2>);
    case 3: return go(k_ms_update_xp<3>);
    case 4: return go(k_ms_update_xp<4>);
    case 5: return go(k_ms_update_xp<5>);
    case 6: return go(k_ms_update_xp<6>);
    case 7: return go(k_ms_update_xp<7>);
    case 8: return go(k_ms_update_xp<8>);
  }
  return hipErrorInvalidValue;
}

}  // namespace wd
