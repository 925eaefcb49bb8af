// CG iterations of a lattice small enough for one workgroup (Vh d_R <= kThreads):
// the recurrence of api.hip with every hop, sum and vector update inside one
// kernel, one block per right-hand side.
//
// A launched iteration of such a lattice is five kernels of 3.5 to 4.5 us that
// hold a block or two each, and the gaps between them: bound by launches and
// latency.  A thread holds one colour of one site, its components of r in
// registers; x, p, u = D-hat p and the odd fields are in LDS (64 KB FP32,
// 128 KB FP64), links come from L2 ahead of the barrier of their hop.  One more
// iteration of a solve (launched: 36 us SU(2), 48 to 100 us with 12 rhs): SU(2)
// FUND 4^4 7.5 us, SU(3) FUND 12.2, SU(2) ADJ 11.4, SU(4) FUND 17.0, and up to
// 3% more with 12 rhs, now bound by the LDS reads (8 d spinor components per
// thread and hop); the solve itself, with its residuals in FP64, takes 140 to
// 156 us (162 to 233 with 12 rhs) whatever the iterations.  Larger lattices fill the LDS or the registers of one CU
// and go back to one launch per hop.  (Twice the threads, each half of them with
// half of the directions: SU(2) 4^4 6% faster, the others 5 to 50% slower.)
#include "wd_common.h"
#include "wd_hop.h"
#include "wd_kernels.h"

namespace wd {

constexpr int kThreads = 512;

struct TinyArgs {
  void *x, *p, *r;        // packed even half fields in T
  const void *links;
  Geom g;
  CgScalars *sc;
  double m4, delta;       // (4 + m0)^2, reliable-update trigger
  int nit;                // iterations at most
};

// Component k of a field in LDS starts at k * pitch<D>(): a constant, so that one
// address a neighbour reads all of its components.
template <int D>
__device__ __forceinline__ constexpr int pitch() {
  return kThreads / D;
}

template <int D, bool REAL, typename T, int MU, int SIG, bool BWD>
__device__ __forceinline__ void tiny_dir(cplx<T> (&acc)[4], const cplx<T> *in,
                                         const typename LinkT<T, REAL>::type (&u)[D]) {
  cplx<T> chi[2] = {mk<T>(0, 0), mk<T>(0, 0)};
#pragma unroll
  for (int b = 0; b < D; ++b) {
    cplx<T> p[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) p[s] = in[(s * D + b) * pitch<D>()];
    chi[0] = link_mac(u[b], p[0] + ipow<PROJ_PH(MU, SIG, 0)>(p[2 + ECOL(MU, 0)]), chi[0], BWD);
    chi[1] = link_mac(u[b], p[1] + ipow<PROJ_PH(MU, SIG, 1)>(p[2 + ECOL(MU, 1)]), chi[1], BWD);
  }
  acc[0] = acc[0] + chi[0];
  acc[1] = acc[1] + chi[1];
  acc[2] = acc[2] + ipow<RECON_PH(MU, SIG, 0)>(chi[RECON_SRC(MU, 0)]);
  acc[3] = acc[3] + ipow<RECON_PH(MU, SIG, 1)>(chi[RECON_SRC(MU, 1)]);
}

// The next direction's reads wait for this one's sums (the scheduler otherwise
// issues all of a hop's reads first: 8 d spinor components, all spilled).
template <typename T>
__device__ __forceinline__ void tiny_next(cplx<T> (&acc)[4], int &j) {
#pragma unroll
  for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(j) : "v"(acc[s].re), "v"(acc[s].im));
}

// acc = -2 H in for the thread's site of parity PAR and colour row; the links
// are loaded ahead of the barrier behind which `in` is complete.  The compiler
// takes the indices as new in each hop: it would otherwise move the addresses
// and loads of all four hops out of the iteration loop and spill them.
template <int D, bool REAL, typename T, int PAR, bool DAG>
__device__ __forceinline__ void tiny_hop(cplx<T> (&acc)[4], const cplx<T> *in,
                                         const typename LinkT<T, REAL>::type *links, int stride, int site, int row,
                                         const int (&nbf)[4], const int (&nbb)[4]) {
  using L = typename LinkT<T, REAL>::type;
  constexpr int E = D * D;
  L uf[4][D], ub[4][D];
  asm volatile("" : "+v"(site), "+v"(row));
  int jf[4], jb[4];
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    jf[mu] = nbf[mu];
    jb[mu] = nbb[mu];
    asm volatile("" : "+v"(jf[mu]), "+v"(jb[mu]));
  }
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    const L *lf = links + (size_t)(PAR * 4 + mu) * E * stride, *lb = links + (size_t)((1 - PAR) * 4 + mu) * E * stride;
    const uint32_t of = (uint32_t)(link_site(E, stride, site) + link_row(row * D, stride)),
                   ob = (uint32_t)(link_site(E, stride, jb[mu]) + link_row(row, stride));
#pragma unroll
    for (int b = 0; b < D; ++b) {
      uf[mu][b] = *at(lf + link_row(b, stride), of);
      ub[mu][b] = *at(lb + link_row(b * D, stride), ob);
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = mk<T>(0, 0);
  constexpr int SF = DAG ? -1 : 1;
  tiny_dir<D, REAL, T, 0, SF, false>(acc, in + jf[0], uf[0]);
  tiny_next(acc, jb[0]);
  tiny_dir<D, REAL, T, 0, -SF, true>(acc, in + jb[0], ub[0]);
  tiny_next(acc, jf[1]);
  tiny_dir<D, REAL, T, 1, SF, false>(acc, in + jf[1], uf[1]);
  tiny_next(acc, jb[1]);
  tiny_dir<D, REAL, T, 1, -SF, true>(acc, in + jb[1], ub[1]);
  tiny_next(acc, jf[2]);
  tiny_dir<D, REAL, T, 2, SF, false>(acc, in + jf[2], uf[2]);
  tiny_next(acc, jb[2]);
  tiny_dir<D, REAL, T, 2, -SF, true>(acc, in + jb[2], ub[2]);
  tiny_next(acc, jf[3]);
  tiny_dir<D, REAL, T, 3, SF, false>(acc, in + jf[3], uf[3]);
  tiny_next(acc, jb[3]);
  tiny_dir<D, REAL, T, 3, -SF, true>(acc, in + jb[3], ub[3]);
}

// Sum over the block in a fixed order, result in every thread; red: one double
// per wavefront, not reused before another barrier.
__device__ __forceinline__ double tiny_sum(double v, double *red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
  return s;
}

template <int D, bool REAL, typename T>
__global__ __launch_bounds__(kThreads) void k_cg_tiny(TinyArgs a) {
  using L = typename LinkT<T, REAL>::type;
  __shared__ cplx<T> ps[4 * kThreads], us[4 * kThreads], os[4 * kThreads], xs[4 * kThreads];   // [component][site]
  __shared__ double red[2][kThreads / 64];
  CgScalars &s = a.sc[blockIdx.x];
  if (!s.active) return;
  const int Vh = a.g.Vh, stride = a.g.stride, n = Vh * D;
  const bool on = (int)threadIdx.x < n;   // the other lanes repeat the last one and store nothing
  const int e = on ? (int)threadIdx.x : n - 1, row = e / Vh, site = e - row * Vh;
  int fe[4], be[4], fo[4], bo[4];   // neighbours of the even and the odd site `site`
  {
    int t, x, y, z;
    cb_coords(a.g, site, 0, t, x, y, z);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      fe[mu] = nb_index(a.g, t, x, y, z, mu, 1);
      be[mu] = nb_index(a.g, t, x, y, z, mu, 0);
    }
    cb_coords(a.g, site, 1, t, x, y, z);
#pragma unroll
    for (int mu = 0; mu < 4; ++mu) {
      fo[mu] = nb_index(a.g, t, x, y, z, mu, 1);
      bo[mu] = nb_index(a.g, t, x, y, z, mu, 0);
    }
  }
  const L *links = static_cast<const L *>(a.links);
  const size_t base = (size_t)blockIdx.x * 4 * D * stride + (size_t)row * stride + site;
  cplx<T> *xg = static_cast<cplx<T> *>(a.x) + base, *pg = static_cast<cplx<T> *>(a.p) + base,
          *rg = static_cast<cplx<T> *>(a.r) + base;
  constexpr int C = D * pitch<D>();   // from one spin to the next
  const int own = on ? row * pitch<D>() + site : 0;
  cplx<T> r[4], v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const size_t o = (size_t)k * D * stride;
    r[k] = rg[o];
    if (on) {
      ps[k * C + own] = pg[o];
      xs[k * C + own] = xg[o];
    }
  }
  double rho = s.rho, rmax = s.rmax, pAp = 0.0, alpha = 0.0;
  const double stop2 = s.stop2;
  int iters = s.iters, status = s.status, active = 1, need = s.need_update;
  const T ca = (T)a.m4, half = (T)0.5;
  for (int it = 0; it < a.nit && active; ++it) {
    // u = D-hat p
    tiny_hop<D, REAL, T, 1, false>(v, ps, links, stride, site, row, fo, bo);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (on) os[k * C + own] = -half * v[k];
    tiny_hop<D, REAL, T, 0, false>(v, os, links, stride, site, row, fe, be);
    double nrm = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const cplx<T> p = ps[k * C + own];
      cplx<T> u = half * v[k];
      u.re = fma(ca, p.re, u.re);
      u.im = fma(ca, p.im, u.im);
      if (on) us[k * C + own] = u;
      nrm += (double)u.re * u.re + (double)u.im * u.im;
    }
    pAp = tiny_sum(on ? nrm : 0.0, red[0]);
    if (!(pAp > 0.0) || !isfinite(pAp) || !isfinite(rho)) {
      status = -5;   // breakdown
      active = 0;
      alpha = 0.0;
      break;
    }
    alpha = rho / pAp;
    // r -= alpha D-hat^+ u
    tiny_hop<D, REAL, T, 1, true>(v, us, links, stride, site, row, fo, bo);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (on) os[k * C + own] = -half * v[k];
    tiny_hop<D, REAL, T, 0, true>(v, os, links, stride, site, row, fe, be);
    nrm = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const cplx<T> u = us[k * C + own];
      cplx<T> q = half * v[k];
      q.re = fma(ca, u.re, q.re);
      q.im = fma(ca, u.im, q.im);
      r[k] = mk<T>((T)fma(-alpha, (double)q.re, (double)r[k].re), (T)fma(-alpha, (double)q.im, (double)r[k].im));
      nrm += (double)r[k].re * r[k].re + (double)r[k].im * r[k].im;
    }
    const double rr = tiny_sum(on ? nrm : 0.0, red[1]);
    // end of the iteration as cg_end_step and k_cg_update_xp (blas.hip)
    ++iters;
    const double b = rr / rho;
    const bool ok = isfinite(rr);
    if (on)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const cplx<T> p = ps[k * C + own], x = xs[k * C + own];
        xs[k * C + own] = mk<T>((T)fma(alpha, (double)p.re, (double)x.re), (T)fma(alpha, (double)p.im, (double)x.im));
        if (ok) ps[k * C + own] = mk<T>((T)fma(b, (double)p.re, (double)r[k].re), (T)fma(b, (double)p.im, (double)r[k].im));
      }
    if (!ok) {
      status = -5;
      active = 0;
      break;
    }
    rho = rr;
    const double rn = sqrt(rr);
    rmax = rn > rmax ? rn : rmax;
    if (rr <= stop2) {
      active = 0;
      need = 1;
    } else if (a.delta > 0.0 && rn < a.delta * rmax) {
      need = 1;
    }
  }
  if (on)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t o = (size_t)k * D * stride;
      xg[o] = xs[k * C + own];
      pg[o] = ps[k * C + own];
      rg[o] = r[k];
    }
  if (threadIdx.x == 0) {
    s.rho = rho;
    s.pAp = pAp;
    s.alpha = alpha;
    s.rmax = rmax;
    s.iters = iters;
    s.status = status;
    s.active = s.act_it = active;
    s.need_update = need;
  }
}

bool cg_tiny_ok(const Geom &g, int d, int real) {
  return (long long)g.Vh * d <= kThreads && (real ? d == 3 : d >= 2 && d <= 4);
}

template <typename T>
static hipError_t launch_t(const TinyArgs &a, int d, int real, int nrhs, hipStream_t st) {
  const dim3 grid(nrhs), block((a.g.Vh * d + 63) / 64 * 64);
  if (real) hipLaunchKernelGGL((k_cg_tiny<3, true, T>), grid, block, 0, st, a);
  else if (d == 2) hipLaunchKernelGGL((k_cg_tiny<2, false, T>), grid, block, 0, st, a);
  else if (d == 3) hipLaunchKernelGGL((k_cg_tiny<3, false, T>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((k_cg_tiny<4, false, T>), grid, block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_cg_tiny(void *x, void *p, void *r, const void *links, const Geom &g, int d, int real, CgScalars *s,
                          double m4, double delta, int nit, int nrhs, int prec, hipStream_t st) {
  if (!cg_tiny_ok(g, d, real)) return hipErrorInvalidValue;
  const TinyArgs a{x, p, r, links, g, s, m4, delta, nit};
  return prec == 0 ? launch_t<double>(a, d, real, nrhs, st) : launch_t<float>(a, d, real, nrhs, st);
}

}  // namespace wd
