// SU(N) matrices in registers and the staging of canonical links
// [T][X][Y][Z][4][N][N] through LDS (hmc.hip).
#pragma once
#include "wd_common.h"

namespace wd {

template <int N>
struct Mat {
  cplx<double> a[N][N];
};

template <int N>
__device__ __forceinline__ Mat<N> ld_mat(const cplx<double> *p, bool dag) {
  Mat<N> m;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const cplx<double> v = p[dag ? j * N + i : i * N + j];
      m.a[i][j] = dag ? mk(v.re, -v.im) : v;
    }
  return m;
}

template <int N>
__device__ __forceinline__ Mat<N> mul(const Mat<N> &x, const Mat<N> &y) {
  Mat<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      cplx<double> s = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < N; ++k) s = cfma(x.a[i][k], y.a[k][j], s);
      r.a[i][j] = s;
    }
  return r;
}

// The loads of LinkTile::fetch() have landed (the caller's barrier makes them visible).
__device__ __forceinline__ void wait_fetch() { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

// Coordinates of lexicographic site lex, and the site one step away along mu.
struct Site {
  int c[4];
  unsigned lex;
  __device__ __forceinline__ Site(const Geom &g, unsigned l) : lex(l) {
    unsigned r = l;
    c[3] = (int)(r % (unsigned)g.Z); r /= (unsigned)g.Z;
    c[2] = (int)(r % (unsigned)g.Y); r /= (unsigned)g.Y;
    c[1] = (int)(r % (unsigned)g.X);
    c[0] = (int)(r / (unsigned)g.X);
  }
  __device__ __forceinline__ int shift(const Geom &g, int mu, int step) const {   // difference of site indices
    const int st = mu == 0 ? g.X * g.Y * g.Z : mu == 1 ? g.Y * g.Z : mu == 2 ? g.Z : 1;
    const int L = mu == 0 ? g.T : mu == 1 ? g.X : mu == 2 ? g.Y : g.Z;
    const int x = mu == 0 ? c[0] : mu == 1 ? c[1] : mu == 2 ? c[2] : c[3];
    const int q = x + step, d = q < 0 ? step + L : q >= L ? step - L : step;
    return d * st;
  }
};

// Block index such that each XCD runs one contiguous range of blocks.
__device__ __forceinline__ unsigned xcd_range(unsigned b, unsigned n) {
  const unsigned q = n >> 3, rmd = n & 7, x = b & 7, j = b >> 3;
  return x * q + (x < rmd ? x : rmd) + j;
}

// off, not known before m is: reads from it are not issued earlier.  (The
// compiler otherwise issues the reads of all steps at once, and spills.)
template <int N>
__device__ __forceinline__ unsigned after(unsigned off, const Mat<N> &m) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+v"(off) : "v"(m.a[i][j].re), "v"(m.a[i][j].im));
  return off;
}

template <int N>
struct Vec {
  cplx<double> a[N];
};

// Links of a tile of S sites that several lanes share, staged through LDS by a
// block of NT threads.  A lane reading its own N^2 entries from the canonical
// layout touches a cache line of its own with every load; here consecutive lanes
// fetch consecutive entries, directly into LDS.  Slot k holds the link
// tab[k S + s] (4 site + direction) of every tile site s in a row of N^2 16-byte
// entries, padded to an odd number: lanes on consecutive sites read without
// bank conflicts.  DIRECT loads take whole 16-byte entries; links whose address is
// not a multiple of 16 go through registers.
inline bool direct_ok(const void *U) { return ((size_t)U & 15) == 0; }
template <int N, int S, int NT, bool DIRECT>
struct LinkTile {
  static constexpr int E = N * N, ROW = E | 1;
  static constexpr int elems(int slots) { return slots * S * ROW; }
  template <int SLOTS>
  static __device__ __forceinline__ void fetch(cplx<double> *buf, const cplx<double> *U, const unsigned *tab) {
    constexpr int n = elems(SLOTS) / 64;   // loads of a wavefront's width
    static_assert(elems(SLOTS) % 64 == 0, "whole loads");
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
#pragma unroll 4
    for (int k = w; k < n; k += NT / 64) {
      const int f = k * 64 + lane, r = f / ROW, q = f - r * ROW, e = q < E ? q : E - 1;
      if constexpr (DIRECT) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(U + (size_t)tab[r] * E + e),
                                         (__attribute__((address_space(3))) void *)(buf + k * 64), 16, 0, 0);
      } else {
        const double *p = reinterpret_cast<const double *>(U) + 2 * ((size_t)tab[r] * E + e);
        buf[f] = mk(p[0], p[1]);
      }
    }
  }
  static __device__ __forceinline__ const cplx<double> *at(const cplx<double> *buf, int slot, int s) {
    return buf + (slot * S + s) * ROW;
  }
};

// Column c of the link at u, of its adjoint, and products with a column.
template <int N>
__device__ __forceinline__ Vec<N> col(const cplx<double> *u, int c) {
  Vec<N> v;
#pragma unroll
  for (int i = 0; i < N; ++i) v.a[i] = u[i * N + c];
  return v;
}
template <int N>
__device__ __forceinline__ Vec<N> col_dag(const cplx<double> *u, int c) {
  Vec<N> v;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const cplx<double> z = u[c * N + i];
    v.a[i] = mk(z.re, -z.im);
  }
  return v;
}
template <int N>
__device__ __forceinline__ Vec<N> mulv(const cplx<double> *u, const Vec<N> &v) {
  Vec<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    r.a[i] = mk(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < N; ++k) r.a[i] = cfma(u[i * N + k], v.a[k], r.a[i]);
  }
  return r;
}
template <int N>
__device__ __forceinline__ Vec<N> mulv_dag(const cplx<double> *u, const Vec<N> &v) {
  Vec<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    r.a[i] = mk(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < N; ++k) r.a[i] = cfma_conj(u[k * N + i], v.a[k], r.a[i]);
  }
  return r;
}
template <int N>
__device__ __forceinline__ void add(Vec<N> &x, const Vec<N> &y) {
#pragma unroll
  for (int i = 0; i < N; ++i) x.a[i] = x.a[i] + y.a[i];
}

}  // namespace wd
