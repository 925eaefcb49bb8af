// Hopping term with a clover block in its epilogue (colour-split form, one
// right-hand side), the two halves of D-hat = D_ee - D_eo D_oo^{-1} D_oe:
//   out = M (beta H in)        (cx NULL: M = D_oo^{-1} on the odd sites), or
//   out = M cx + beta H in     (M = D_ee on the even sites).
//
// As passes of its own a clover block costs 33 us on SU(3) FUND 24^4 (672 bytes
// of matrix and 384 of spinor a site, at the copy rate) beside 52 us for a hop;
// in the epilogue the spinor's two passes are gone (68 us a hop with its
// block, launched back to back).  A wavefront holds one colour row of 64 sites: the rows of the
// vector that M multiplies meet in the hop's LDS, and each lane forms its four
// spins, reading the rows of M it needs from the packed triangle (an entry off
// the diagonal serves two wavefronts of the block, the second through L1 or L2).
#include "wd_hop_cs.h"
#include "wd_kernels.h"

namespace wd {

template <int D, typename T, bool DAG, int STG, int W>
__global__ __launch_bounds__(64 * D) __attribute__((amdgpu_waves_per_eu(W))) void k_hop_clover(HopArgs a) {
  constexpr int NB = 2 * STG, B2 = 2 * D, NT = B2 * (B2 + 1) / 2;
  __shared__ cplx<T> hs[NB][1][2][D][64];
  __shared__ double sh[D];
  if ((int)blockIdx.x < a.lead) return hop_lead(a);
  const int w = tile_of_block(blockIdx.x - a.lead, a.ntiles, a.xcd_remap);
  const int tile = tile_order(w, a);
  const int l = lattice_of_tile(a, tile);
  const Geom g = a.lat[l].g;
  const int tl = tile - a.lat[l].tile0;
  const int lane = threadIdx.x & 63, row = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int i = tl * 64 + lane;
  const bool valid = i < g.Vh;
  const int is = valid ? i : g.Vh - 1;   // lanes past the end: see k_hop_sp
  const size_t fbase = (size_t)a.lat[l].soff, rstride = 0;
  const cplx<T> *in0 = static_cast<const cplx<T> *>(a.in) + fbase;
  const cplx<T> *links = static_cast<const cplx<T> *>(a.links) + a.lat[l].loff;
  int t, x, y, z;
  cb_coords(g, is, a.parity, t, x, y, z);
  cplx<T> acc[1][4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[0][s] = mk<T>(0, 0);
  constexpr int SF = DAG ? -1 : 1;   // forward hop: 1 - g_mu (dagger: 1 + g_mu)
  if constexpr (STG == 4) {
    cs_mu2<D, false, T, 0, SF, 1, true, 0>(acc, hs, g, a.parity, links, nullptr, in0, rstride, t, x, y, z, is, row, lane);
    cs_mu2<D, false, T, 2, SF, 1, true, 0>(acc, hs, g, a.parity, links, nullptr, in0, rstride, t, x, y, z, is, row, lane);
  } else {
    cplx<T>(*fls)[1][64] = nullptr;
    cs_mu<D, false, T, 0, SF, 1, STG, true, NB, 0>(acc, hs, fls, g, a.parity, links, nullptr, in0, rstride, t, x, y, z,
                                                   is, row, lane);
    cs_mu<D, false, T, 1, SF, 1, STG, true, NB, 0>(acc, hs, fls, g, a.parity, links, nullptr, in0, rstride, t, x, y, z,
                                                   is, row, lane);
    cs_mu<D, false, T, 2, SF, 1, STG, true, NB, 0>(acc, hs, fls, g, a.parity, links, nullptr, in0, rstride, t, x, y, z,
                                                   is, row, lane);
    cs_mu<D, false, T, 3, SF, 1, STG, true, NB, 0>(acc, hs, fls, g, a.parity, links, nullptr, in0, rstride, t, x, y, z,
                                                   is, row, lane);
  }
  const T cb = (T)(-0.5 * a.beta);
  const cplx<T> *cx = static_cast<const cplx<T> *>(a.cx);
  cplx<T> v[4];   // beta H in
#pragma unroll
  for (int s = 0; s < 4; ++s) v[s] = cb * acc[0][s];
  __syncthreads();   // every wavefront has read its last projections
  cplx<T>(*ys)[D][64] = &hs[0][0][0];   // the vector that M multiplies, [spin][colour][site]
#pragma unroll
  for (int s = 0; s < 4; ++s)
    ys[s][row][lane] = cx ? ld_nt(cx + fbase + (size_t)(s * D + row) * g.stride + i) : v[s];
  __syncthreads();
  const cplx<T> *M = static_cast<const cplx<T> *>(a.clov) + fbase * (2 * D + 1) +
                     (size_t)a.parity * 2 * NT * g.stride + is;
  cplx<T> o[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int c = s >> 1, h = s & 1, r = h * D + row;   // row r of block c
    cplx<T> e[B2];
#pragma unroll
    for (int j = 0; j < B2; ++j) {
      const int lo = r < j ? r : j, hi = r < j ? j : r;
      e[j] = M[(size_t)(c * NT + lo * B2 - lo * (lo - 1) / 2 + hi - lo) * g.stride];
      if (j < h * D) e[j].im = -e[j].im;
      else if (j < h * D + D) e[j].im = r > j ? -e[j].im : e[j].im;
    }
    cplx<T> q = mk<T>(0, 0);
#pragma unroll
    for (int j = 0; j < B2; ++j) q = cfma(e[j], ys[2 * c + j / D][j % D][lane], q);
    o[s] = q;
    if (s == 1) __builtin_amdgcn_sched_barrier(0);   // one block's entries at a time
  }
  if (cx)
#pragma unroll
    for (int s = 0; s < 4; ++s) o[s] = o[s] + v[s];
  double nrm = 0.0;
  if (a.r) {
    cplx<T> *rf = static_cast<cplx<T> *>(a.r) + fbase;
    const cplx<T> *ri = static_cast<const cplx<T> *>(a.rin) + fbase, *ps = static_cast<const cplx<T> *>(a.ps) + fbase;
    const RStep<T> step(a, l);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const size_t k = (size_t)(s * D + row) * g.stride + i;
      const cplx<T> rn = step(rf + k, ld_nt(ri + k), ps + k, o[s]);
      nrm += (double)rn.re * rn.re + (double)rn.im * rn.im;
    }
  } else {
    cplx<T> *out = static_cast<cplx<T> *>(a.out) + fbase;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      st_nt(out + (size_t)(s * D + row) * g.stride + i, o[s]);
      nrm += (double)o[s].re * o[s].re + (double)o[s].im * o[s].im;
    }
  }
  if (a.partial) {
    const double p = block_sum(valid ? nrm : 0.0, sh);
    if (threadIdx.x == 0) a.partial[(size_t)l * a.prow + tl] = p;
  }
}

bool hop_clover_ok(int d, int variant) {
  return d >= 2 && d <= 4 && (variant == HOP_COLOUR || variant == HOP_COLOUR_PAIR || variant == HOP_COLOUR_QUAD);
}

template <int D, typename T, bool DAG>
static hipError_t launch_d(HopArgs a, int variant, hipStream_t st) {
  constexpr int W = cs_waves(D, sizeof(T) == 8, 1);
  const dim3 grid(a.ntiles + a.lead);
  if (variant == HOP_COLOUR_QUAD)
    hipLaunchKernelGGL((k_hop_clover<D, T, DAG, 4, W>), grid, dim3(64 * D), 0, st, a);
  else if (variant == HOP_COLOUR_PAIR)
    hipLaunchKernelGGL((k_hop_clover<D, T, DAG, 2, W>), grid, dim3(64 * D), 0, st, a);
  else
    hipLaunchKernelGGL((k_hop_clover<D, T, DAG, 1, W>), grid, dim3(64 * D), 0, st, a);
  return hipGetLastError();
}

template <typename T, bool DAG>
static hipError_t launch_t(const HopArgs &a, int d, int variant, hipStream_t st) {
  return d == 2 ? launch_d<2, T, DAG>(a, variant, st)
       : d == 3 ? launch_d<3, T, DAG>(a, variant, st)
                : launch_d<4, T, DAG>(a, variant, st);
}

hipError_t launch_hop_clover(const HopArgs &a0, int d, int prec, int dagger, int variant, hipStream_t st,
                             Counts *counts, int *prow) {
  if (!hop_clover_ok(d, variant)) return hipErrorInvalidValue;
  HopArgs a = a0;
  set_tiles(a, 64, 1, counts, prow);
  a.ngroups = 1;
  if (prec == 0) return dagger ? launch_t<double, true>(a, d, variant, st) : launch_t<double, false>(a, d, variant, st);
  return dagger ? launch_t<float, true>(a, d, variant, st) : launch_t<float, false>(a, d, variant, st);
}

}  // namespace wd
