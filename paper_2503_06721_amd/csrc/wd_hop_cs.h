// Building blocks of the colour-split hopping term: staging, compute and phase
// order of k_hop_cs (hop.hip) and k_hop_clover (hop_clover.hip).
#pragma once
#include "wd_common.h"
#include "wd_hop.h"
#include "wd_rep.h"

namespace wd {

// Stage: this lane's link entries (row `row` of U for a forward hop, column
// `row` of U for a backward hop, whose U^+ row is the conjugated column) and
// colour component `row` of the neighbour spinor, spin-projected into LDS.
//
// Compact form (FLY = 2 SYM, 3 2AS): the entries are rebuilt from the
// fundamental link, (U_R)_AB = n_A n_B (U_ac U_bd +- U_ad U_bc) with
// (a, b) = pair(A), (c, d) = pair(B), n = 1/sqrt2 on the diagonal pairs of
// SYM and 1 otherwise -- the closed forms of wd_rep.h.  Row `row` of U_R needs
// the fundamental rows a, b; column `row` (backward hop) the columns a, b.
// The boundary phase is stored as i U (the maps are quadratic).
template <int D, bool SYM>
constexpr int two_index_n() {
  return SYM ? (D == 3 ? 2 : D == 6 ? 3 : 4) : (D == 3 ? 3 : D == 6 ? 4 : 5);
}

// First and second index of two-index basis element A, at compile time.
constexpr int pair_first(int N, bool SYM, int A) {
  int a = 0, rem = A;
  while (rem >= (SYM ? N - a : N - 1 - a)) {
    rem -= SYM ? N - a : N - 1 - a;
    ++a;
  }
  return a;
}
constexpr int pair_second(int N, bool SYM, int A) {
  int a = 0, rem = A;
  while (rem >= (SYM ? N - a : N - 1 - a)) {
    rem -= SYM ? N - a : N - 1 - a;
    ++a;
  }
  return a + rem + (SYM ? 0 : 1);
}

// u[B] = nA nB (x[c] y[d] +- x[d] y[c]), (c, d) = pair(B), unrolled over B so
// that every register index is a constant.
template <int D, int N, bool SYM, typename T, int B = 0>
__device__ __forceinline__ void rebuild_row(cplx<T> (&u)[D], const cplx<T> (&xr)[N], const cplx<T> (&yr)[N], T na) {
  if constexpr (B < D) {
    constexpr int c = pair_first(N, SYM, B), d = pair_second(N, SYM, B);
    const T nn = (SYM && c == d) ? na * (T)0.70710678118654752440 : na;
    const cplx<T> p = cmul(xr[c], yr[d]), q = cmul(xr[d], yr[c]);
    u[B] = SYM ? mk<T>(nn * (p.re + q.re), nn * (p.im + q.im)) : mk<T>(nn * (p.re - q.re), nn * (p.im - q.im));
    rebuild_row<D, N, SYM, T, B + 1>(u, xr, yr, na);
  }
}

// Fundamental entries per link of the compact form FLY (1 for stored links),
// and the LDS rows that hold them: a multiple of D, so that every wave loads
// the same number of entries (the last rows repeat entry NE - 1 unused).
template <int D, int FLY>
constexpr int fly_entries() {
  return FLY ? two_index_n<D, FLY == 2>() * two_index_n<D, FLY == 2>() : 1;
}
template <int D, int FLY>
constexpr int fly_rows() {
  return FLY ? (fly_entries<D, FLY>() + D - 1) / D * D : 1;
}

// Stage one hop.  Stored links: this lane's row (forward) or column
// (backward) of U_R into registers u.  Compact form: the block's waves share
// the N^2 fundamental entries of each site's link, wave `row` loading entries
// row, row + D, ... into fl (each entry is read from memory once per site, not
// once per wave that needs it); u is rebuilt from fl after the barrier
// (cs_rebuild).  Then the spin projection of colour `row` of the neighbour
// spinor into hs.
template <int D, bool REAL, typename T, int MU, int SIG, bool BWD, int NR, bool NTL, int FLY>
__device__ __forceinline__ void cs_stage(typename LinkT<T, REAL>::type (&u)[D], cplx<T> (*hs)[2][D][64],
                                         cplx<T> (*fl)[64], const Geom &g, int parity,
                                         const typename LinkT<T, REAL>::type *links, const cplx<T> *flinks,
                                         const cplx<T> *in0, size_t rstride, int nb, int lsite, int row, int lane) {
  using L = typename LinkT<T, REAL>::type;
  const int stride = g.stride;
  const int lpar = BWD ? 1 - parity : parity;
  if constexpr (FLY != 0) {
    constexpr int NE = fly_entries<D, FLY>();
    const cplx<T> *fk = flinks + (size_t)(lpar * 4 + MU) * NE * stride + link_site(NE, stride, lsite);
#pragma unroll
    for (int j = 0; j < fly_rows<D, FLY>() / D; ++j) {
      const int e = row + j * D;
      fl[e][lane] = ld_stream<NTL>(fk + link_row(e < NE ? e : NE - 1, stride));
    }
  } else {
    const L *lk = links + (size_t)(lpar * 4 + MU) * D * D * stride;
#pragma unroll
    for (int b = 0; b < D; ++b)
      u[b] = ld_stream<NTL>(lk + link_row(BWD ? b * D + row : row * D + b, stride) + link_site(D * D, stride, lsite));
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const cplx<T> *in = in0 + k * rstride;
    cplx<T> p[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) p[s] = in[(size_t)(s * D + row) * stride + nb];
    hs[k][0][row][lane] = p[0] + ipow<PROJ_PH(MU, SIG, 0)>(p[2 + ECOL(MU, 0)]);
    hs[k][1][row][lane] = p[1] + ipow<PROJ_PH(MU, SIG, 1)>(p[2 + ECOL(MU, 1)]);
  }
}

// Compact form, after the barrier: rebuild this lane's row (forward) or
// column (backward) of U_R from the fundamental rows (columns) a1, a2 staged
// in fl.
// (No-op for stored links.)
template <int D, typename T, bool BWD, int FLY, typename U>
__device__ __forceinline__ void cs_rebuild(U (&u)[D], cplx<T> (*fl)[64], int row, int lane) {
  if constexpr (FLY != 0) {
    constexpr bool SYM = FLY == 2;
    constexpr int N = two_index_n<D, SYM>();
    int a1, a2;
    pair_of<N, SYM>(row, a1, a2);
    cplx<T> xr[N], yr[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      xr[c] = fl[BWD ? c * N + a1 : a1 * N + c][lane];
      yr[c] = fl[BWD ? c * N + a2 : a2 * N + c][lane];
    }
    rebuild_row<D, N, SYM, T>(u, xr, yr, (SYM && a1 == a2) ? (T)0.70710678118654752440 : (T)1);
  }
}

// Compute: after the barrier, the full projected two-spinor of this lane's
// site is in LDS; apply the link row and reconstruct the lower spin half.
template <int D, bool REAL, typename T, int MU, int SIG, bool BWD, int NR>
__device__ __forceinline__ void cs_compute(cplx<T> (&acc)[NR][4], const typename LinkT<T, REAL>::type (&u)[D],
                                           cplx<T> (*hs)[2][D][64], int lane) {
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    cplx<T> chi[2] = {mk<T>(0, 0), mk<T>(0, 0)};
#pragma unroll
    for (int b = 0; b < D; ++b) {
      chi[0] = link_mac(u[b], hs[k][0][b][lane], chi[0], BWD);
      chi[1] = link_mac(u[b], hs[k][1][b][lane], chi[1], BWD);
    }
    acc[k][0] = acc[k][0] + chi[0];
    acc[k][1] = acc[k][1] + chi[1];
    acc[k][2] = acc[k][2] + ipow<RECON_PH(MU, SIG, 0)>(chi[RECON_SRC(MU, 0)]);
    acc[k][3] = acc[k][3] + ipow<RECON_PH(MU, SIG, 1)>(chi[RECON_SRC(MU, 1)]);
  }
  // keep each phase's arithmetic next to its barrier
  __builtin_amdgcn_sched_barrier(0);
}

// One direction mu.  STG = 1: forward and backward hops are two barrier
// phases (LDS buffers 0 and 1).  STG = 2: both are staged before a single
// barrier (LDS buffers 2*(MU&1) and 2*(MU&1)+1), which halves the barriers and
// doubles the loads in flight per phase at the cost of twice the LDS.
// (STG = 4, two directions per phase, is cs_mu2 below.)
template <int D, bool REAL, typename T, int MU, int SF, int NR, int STG, bool NTL, int NB, int FLY>
__device__ __forceinline__ void cs_mu(cplx<T> (&acc)[NR][4], cplx<T> (*hs)[NR][2][D][64],
                                      cplx<T> (*fls)[(fly_rows<D, FLY>())][64], const Geom &g, int parity,
                                      const typename LinkT<T, REAL>::type *links, const cplx<T> *flinks,
                                      const cplx<T> *in0, size_t rstride, int t, int x, int y, int z, int is, int row,
                                      int lane) {
  using L = typename LinkT<T, REAL>::type;
  const int nbf = nb_index(g, t, x, y, z, MU, 1);
  const int nbb = nb_index(g, t, x, y, z, MU, 0);
  L uf[D], ub[D];
  if constexpr (STG == 2) {
    constexpr int B0 = 2 * (MU & 1);
    cs_stage<D, REAL, T, MU, SF, false, NR, NTL, FLY>(uf, hs[B0], fls[B0], g, parity, links, flinks, in0, rstride,
                                                      nbf, is, row, lane);
    cs_stage<D, REAL, T, MU, -SF, true, NR, NTL, FLY>(ub, hs[B0 + 1], fls[B0 + 1], g, parity, links, flinks, in0,
                                                      rstride, nbb, nbb, row, lane);
    __syncthreads();
    cs_rebuild<D, T, false, FLY>(uf, fls[B0], row, lane);
    cs_compute<D, REAL, T, MU, SF, false, NR>(acc, uf, hs[B0], lane);
    cs_rebuild<D, T, true, FLY>(ub, fls[B0 + 1], row, lane);
    cs_compute<D, REAL, T, MU, -SF, true, NR>(acc, ub, hs[B0 + 1], lane);
  } else {
    cs_stage<D, REAL, T, MU, SF, false, NR, NTL, FLY>(uf, hs[0], fls[0], g, parity, links, flinks, in0, rstride, nbf,
                                                      is, row, lane);
    __syncthreads();
    cs_rebuild<D, T, false, FLY>(uf, fls[0], row, lane);
    cs_compute<D, REAL, T, MU, SF, false, NR>(acc, uf, hs[0], lane);
    cs_stage<D, REAL, T, MU, -SF, true, NR, NTL, FLY>(ub, hs[1], fls[1], g, parity, links, flinks, in0,
                                                      rstride, nbb, nbb, row, lane);
    __syncthreads();
    cs_rebuild<D, T, true, FLY>(ub, fls[1], row, lane);
    cs_compute<D, REAL, T, MU, -SF, true, NR>(acc, ub, hs[1], lane);
  }
}

// Compact form, software-pipelined (FP64, one rhs per block, STG = 1): the
// global loads of hop h + 1 (this wave's fundamental link entries and spinor
// components) are issued right after hop h's barrier and land while hop h
// rebuilds its link row and computes; one barrier per hop over the two LDS
// buffer sets (a buffer is rewritten two hops after it was read, with a
// barrier between).  Measured per hop: SU(3) SYM 48x24^3 212 -> 191 us,
// SU(4) 2AS 96x48^3 4769 -> 4014 us; in FP32 it gains nothing (1811 -> 1859
// us for SU(4) 2AS) and is not used.
template <int D, typename T, int NR, int FLY>
struct CsRaw {
  cplx<T> f[fly_rows<D, FLY>() / D];   // fundamental entries row, row + D, ...
  cplx<T> p[NR][4];                     // colour `row` of the neighbour spinor, per spin
};

template <int D, typename T, int MU, bool BWD, int NR, bool NTL, int FLY>
__device__ __forceinline__ void cs_load(CsRaw<D, T, NR, FLY> &rw, const Geom &g, int parity, const cplx<T> *flinks,
                                        const cplx<T> *in0, size_t rstride, int nb, int lsite, int row) {
  constexpr int NE = fly_entries<D, FLY>();
  const int stride = g.stride;
  const int lpar = BWD ? 1 - parity : parity;
  const cplx<T> *fk = flinks + (size_t)(lpar * 4 + MU) * NE * stride + link_site(NE, stride, lsite);
#pragma unroll
  for (int j = 0; j < fly_rows<D, FLY>() / D; ++j) {
    const int e = row + j * D;
    rw.f[j] = ld_stream<NTL>(fk + link_row(e < NE ? e : NE - 1, stride));
  }
#pragma unroll
  for (int k = 0; k < NR; ++k)
#pragma unroll
    for (int s = 0; s < 4; ++s) rw.p[k][s] = in0[k * rstride + (size_t)(s * D + row) * stride + nb];
}

template <int D, typename T, int MU, int SIG, int NR, int FLY>
__device__ __forceinline__ void cs_publish(const CsRaw<D, T, NR, FLY> &rw, cplx<T> (*hs)[2][D][64], cplx<T> (*fl)[64],
                                           int row, int lane) {
#pragma unroll
  for (int j = 0; j < fly_rows<D, FLY>() / D; ++j) fl[row + j * D][lane] = rw.f[j];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    hs[k][0][row][lane] = rw.p[k][0] + ipow<PROJ_PH(MU, SIG, 0)>(rw.p[k][2 + ECOL(MU, 0)]);
    hs[k][1][row][lane] = rw.p[k][1] + ipow<PROJ_PH(MU, SIG, 1)>(rw.p[k][2 + ECOL(MU, 1)]);
  }
}

template <int D, typename T, int SF, int NR, bool NTL, int FLY, int H = 0>
__device__ __forceinline__ void cs_pipe(cplx<T> (&acc)[NR][4], cplx<T> (*hs)[NR][2][D][64],
                                        cplx<T> (*fls)[(fly_rows<D, FLY>())][64], CsRaw<D, T, NR, FLY> &rw,
                                        const Geom &g, int parity, const cplx<T> *flinks, const cplx<T> *in0,
                                        size_t rstride, const int (&nbf)[4], const int (&nbb)[4], int is, int row,
                                        int lane) {
  if constexpr (H < 8) {
    constexpr int MU = H / 2;
    constexpr bool BWD = (H & 1) != 0;
    constexpr int SIG = BWD ? -SF : SF;
    cs_publish<D, T, MU, SIG, NR, FLY>(rw, hs[H & 1], fls[H & 1], row, lane);
    __syncthreads();
    if constexpr (H < 7) {
      constexpr int MU1 = (H + 1) / 2;
      constexpr bool BWD1 = ((H + 1) & 1) != 0;
      cs_load<D, T, MU1, BWD1, NR, NTL, FLY>(rw, g, parity, flinks, in0, rstride, BWD1 ? nbb[MU1] : nbf[MU1],
                                             BWD1 ? nbb[MU1] : is, row);
    }
    cplx<T> u[D];
    cs_rebuild<D, T, BWD, FLY>(u, fls[H & 1], row, lane);
    cs_compute<D, false, T, MU, SIG, BWD, NR>(acc, u, hs[H & 1], lane);
    cs_pipe<D, T, SF, NR, NTL, FLY, H + 1>(acc, hs, fls, rw, g, parity, flinks, in0, rstride, nbf, nbb, is, row,
                                           lane);
  }
}

// Directions MU0 and MU0 + 1 together (STG = 4): the four hops are staged
// into LDS buffers 2*MU0 .. 2*MU0 + 3 before one barrier, so a launch has two
// barrier phases and four hops' loads in flight in each.
template <int D, bool REAL, typename T, int MU0, int SF, int NR, bool NTL, int FLY>
__device__ __forceinline__ void cs_mu2(cplx<T> (&acc)[NR][4], cplx<T> (*hs)[NR][2][D][64], const Geom &g, int parity,
                                       const typename LinkT<T, REAL>::type *links, const cplx<T> *flinks,
                                       const cplx<T> *in0, size_t rstride, int t, int x, int y, int z, int is, int row,
                                       int lane) {
  using L = typename LinkT<T, REAL>::type;
  constexpr int MU1 = MU0 + 1, B0 = 2 * MU0;
  const int f0 = nb_index(g, t, x, y, z, MU0, 1), b0 = nb_index(g, t, x, y, z, MU0, 0);
  const int f1 = nb_index(g, t, x, y, z, MU1, 1), b1 = nb_index(g, t, x, y, z, MU1, 0);
  static_assert(FLY == 0, "four hops per phase: stored links only");
  L u0f[D], u0b[D], u1f[D], u1b[D];
  cs_stage<D, REAL, T, MU0, SF, false, NR, NTL, 0>(u0f, hs[B0], nullptr, g, parity, links, flinks, in0, rstride, f0,
                                                   is, row, lane);
  cs_stage<D, REAL, T, MU0, -SF, true, NR, NTL, 0>(u0b, hs[B0 + 1], nullptr, g, parity, links, flinks, in0, rstride,
                                                   b0, b0, row, lane);
  cs_stage<D, REAL, T, MU1, SF, false, NR, NTL, 0>(u1f, hs[B0 + 2], nullptr, g, parity, links, flinks, in0, rstride,
                                                   f1, is, row, lane);
  cs_stage<D, REAL, T, MU1, -SF, true, NR, NTL, 0>(u1b, hs[B0 + 3], nullptr, g, parity, links, flinks, in0, rstride,
                                                   b1, b1, row, lane);
  __syncthreads();
  cs_compute<D, REAL, T, MU0, SF, false, NR>(acc, u0f, hs[B0], lane);
  cs_compute<D, REAL, T, MU0, -SF, true, NR>(acc, u0b, hs[B0 + 1], lane);
  cs_compute<D, REAL, T, MU1, SF, false, NR>(acc, u1f, hs[B0 + 2], lane);
  cs_compute<D, REAL, T, MU1, -SF, true, NR>(acc, u1b, hs[B0 + 3], lane);
}

// Waves per SIMD the register allocator is asked to allow (VGPR budget
// 512 / W per lane), chosen per (d_R, precision, right-hand sides per block)
// as the largest value that compiles without spills for the colour-split
// kernel.  (d_R = 15 is capped at 128 VGPRs by its 960-lane block and
// spills a little.)
constexpr int cs_waves(int D, bool dbl, int NR) {
  const int w = dbl ? (D <= 3 ? 4 : D <= 8 ? 3 : 2) : (D <= 4 ? 6 : D <= 6 ? 5 : D <= 10 ? 4 : 3);
  const int cut = NR >= 6 ? 3 : NR >= 3 ? 2 : NR == 2 ? 1 : 0;
  return w - cut > 1 ? w - cut : 1;
}
constexpr int sp_waves(int D, bool dbl) { return dbl ? 2 : (D <= 2 ? 4 : D <= 4 ? 2 : 3); }
// LDS of one colour-split block, hs[NB][NR][2][D][64], must fit the 160 KB
// a gfx950 workgroup may allocate (less the reduction scratch).  Blocks above
// 80 KB run one per CU; the autotuner weighs that against the link sharing.
constexpr int LDS_BUDGET = 160 * 1024 - 256;
template <int D, typename T, int NR, int STG, int FLY = 0>
constexpr bool cs_fits() {
  return 2 * STG * (NR * 2 * D + (FLY ? fly_rows<D, FLY>() : 0)) * 64 * (int)sizeof(cplx<T>) <= LDS_BUDGET;
}

}  // namespace wd
