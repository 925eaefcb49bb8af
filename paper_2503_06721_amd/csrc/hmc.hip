// Gauge-field pieces of the HMC molecular dynamics (Sec. 5.2, 5.3), on the
// caller's canonical fundamental links U [T][X][Y][Z][4][N][N] and momenta pi
// of the same layout (Hermitian traceless matrices pi = pi^a T^a):
//  * Wilson plaquette action S_g = beta sum_x sum_{mu<nu} (1 - Re tr P / N),
//  * its force F = sum_a (dS_g/dw^a) T^a for U -> exp(i w^a T^a) U,
//    dS_g/dw^a_mu(x) = (beta/N) Im tr(T^a U_mu(x) A_mu(x)), A the staple sum,
//    which with B = (M - M^+)/(2i), M = U A, is (beta/N) (B - tr B / N)/2,
//  * the link update U <- exp(i eps pi) U and the kinetic term sum tr(pi^2).
#include "wd_common.h"
#include "wd_kernels.h"

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
__device__ __forceinline__ Mat<N> dagger(const Mat<N> &x) {
  Mat<N> r;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) r.a[i][j] = mk(x.a[j][i].re, -x.a[j][i].im);
  return r;
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

// Links of the 64 lanes of a wavefront, staged through LDS.  A lane reading its
// own N^2 entries from the canonical layout touches a cache line of its own
// with every load: 64 lines a load, the bound of these kernels before.  Here
// consecutive lanes fetch consecutive entries (lane's flat index k 64 + lane =
// entry f % N^2 of the link of lane f / N^2), directly into LDS, where each
// lane then finds its link (N^2 16-byte entries in a row).
template <int N>
struct LinkStage {
  static constexpr int E = N * N, ELEMS = 64 * E;   // entries of one buffer
  // buf <- link (site, mu) of every lane (32-bit site index)
  static __device__ __forceinline__ void fetch(cplx<double> *buf, const cplx<double> *U, unsigned site, int mu) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int f = k * 64 + lane, m = f / E, e = f - m * E;
      const unsigned s = (unsigned)__shfl((int)site, m, 64);
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(U + ((size_t)s * 4 + mu) * E + e),
          (__attribute__((address_space(3))) void *)(buf + k * 64), 16, 0, 0);
    }
  }
  static __device__ __forceinline__ Mat<N> read(const cplx<double> *buf, bool dag) {
    return ld_mat<N>(buf + (threadIdx.x & 63) * E, dag);
  }
};
// The loads of fetch() have landed (the caller's barrier makes them visible).
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

// F = scale * (beta/N) (B - tr B/N)/2 (+ F) per link.  One wavefront per block:
// 64 consecutive sites and one direction mu, the four directions of 64 sites
// in consecutive blocks of one XCD.  The three links of a staple are staged
// while the staple before is multiplied.  SU(3) 24^4: 493 us with a lane
// reading its own links, 406 us; bound by the latency of the staged loads (19 a
// link, 27 KB of LDS a wavefront, five wavefronts a CU).
template <int N>
__global__ __launch_bounds__(64) void k_gauge_force(const cplx<double> *__restrict__ U, cplx<double> *F, Geom g,
                                                    double beta, double scale, int accumulate) {
  using LS = LinkStage<N>;
  __shared__ cplx<double> buf[3][LS::ELEMS];
  const unsigned V = 2 * (unsigned)g.Vh;
  const unsigned b = xcd_range(blockIdx.x, gridDim.x);
  const int mu = (int)(b & 3), lane = threadIdx.x;
  const unsigned lex = (b >> 2) * 64 + lane;
  const Site x(g, lex < V ? lex : V - 1);   // lanes past the end repeat the last site and store nothing
  const unsigned xp = x.lex + x.shift(g, mu, 1);
  Mat<N> A;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) A.a[i][j] = mk(0.0, 0.0);
  // staple s: direction nu = the (s / 2)-th other than mu, upper (s even):
  //   U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
  // lower: U_nu(x+mu-nu)^+ U_mu(x-nu)^+ U_nu(x-nu)
  const auto stage = [&](int s) {
    const int nu = (s >> 1) + ((s >> 1) >= mu), low = s & 1;
    const int d = x.shift(g, nu, low ? -1 : 1);
    LS::fetch(buf[0], U, low ? xp + d : xp, nu);
    LS::fetch(buf[1], U, x.lex + d, mu);
    LS::fetch(buf[2], U, low ? x.lex + d : x.lex, nu);
  };
  stage(0);
#pragma unroll 1
  for (int s = 0; s < 6; ++s) {
    wait_fetch();
    __syncthreads();
    const bool low = s & 1;
    Mat<N> l0 = LS::read(buf[0], false), l2 = LS::read(buf[2], false);
    const Mat<N> l1 = LS::read(buf[1], true);
    __syncthreads();
    if (s < 5) stage(s + 1);
    else LS::fetch(buf[0], U, x.lex, mu);
    if (low) l0 = dagger(l0);
    else l2 = dagger(l2);
    const Mat<N> m = mul<N>(mul<N>(l0, l1), l2);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) A.a[i][j] = A.a[i][j] + m.a[i][j];
  }
  wait_fetch();
  __syncthreads();
  const Mat<N> M = mul<N>(LS::read(buf[0], false), A);
  // B = (M - M^+)/(2i): B_ij = (M_ij - conj(M_ji)) / (2i)
  double trB = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) trB += M.a[i][i].im;
  const double c = scale * beta / N * 0.5;
  cplx<double> *own = buf[1] + lane * LS::E;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double re = M.a[i][j].re - M.a[j][i].re, im = M.a[i][j].im + M.a[j][i].im;
      own[i * N + j] = mk(c * (0.5 * im - (i == j ? trB / N : 0.0)), c * (-0.5 * re));
    }
  __syncthreads();
  const unsigned n = V - (b >> 2) * 64 < 64 ? V - (b >> 2) * 64 : 64;   // links of this block
#pragma unroll
  for (int k = 0; k < LS::E; ++k) {
    const unsigned f = k * 64 + lane, m = f / LS::E, e = f - m * LS::E;
    if (m < n) {
      cplx<double> *out = F + (((size_t)(b >> 2) * 64 + m) * 4 + mu) * LS::E + e;
      cplx<double> v = buf[1][f];
      if (accumulate) v = v + *out;
      *out = v;
    }
  }
}

// Sum over the sites of Re tr P_mu,nu / N over the six planes; a partial sum
// per block of 64 sites, whose three wavefronts take two planes each.  tr P =
// sum_ij a_ij conj(b_ij), a = U_mu(x) U_nu(x+mu), b = U_nu(x) U_mu(x+nu), links
// staged as above.  SU(3) 24^4: 336 us before, 116 us.
template <int N>
__global__ __launch_bounds__(192) void k_plaquette_partial(const cplx<double> *__restrict__ U, double *partial,
                                                           Geom g) {
  using LS = LinkStage<N>;
  __shared__ cplx<double> buf[3][2][LS::ELEMS];
  __shared__ double sh[3];
  const unsigned V = 2 * (unsigned)g.Vh;
  const unsigned blk = xcd_range(blockIdx.x, gridDim.x);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const unsigned lex = blk * 64 + (threadIdx.x & 63);
  const Site x(g, lex < V ? lex : V - 1);
  double s = 0.0;
#pragma unroll 1
  for (int q = 0; q < 2; ++q) {
    const int p = 2 * w + q;   // (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
    const int mu = p < 3 ? 0 : p < 5 ? 1 : 2, nu = p < 3 ? p + 1 : p < 5 ? p - 1 : 3;
    Mat<N> a;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m = h ? nu : mu, n = h ? mu : nu;
      LS::fetch(buf[w][0], U, x.lex, m);
      LS::fetch(buf[w][1], U, x.lex + x.shift(g, m, 1), n);
      wait_fetch();
      __syncthreads();
      const Mat<N> r = mul<N>(LS::read(buf[w][0], false), LS::read(buf[w][1], false));
      __syncthreads();
      if (h == 0) {
        a = r;
      } else {
        double tr = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int j = 0; j < N; ++j) {
            tr = fma(a.a[i][j].re, r.a[i][j].re, tr);
            tr = fma(a.a[i][j].im, r.a[i][j].im, tr);
          }
        s += tr / N;
      }
    }
  }
  s = block_sum(lex < V ? s : 0.0, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// Thread per link: U <- exp(i eps pi) U, the exponential by scaling and
// squaring of its Taylor series (degree 16 after scaling below 1/4).
template <int N>
__global__ __launch_bounds__(256) void k_link_update(cplx<double> *U, const cplx<double> *__restrict__ pi, Geom g,
                                                     double eps) {
  const size_t V = 2 * (size_t)g.Vh;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= 4 * V) return;
  Mat<N> X;   // i eps pi
  double nrm = 0.0;
  const cplx<double> *p = pi + gid * N * N;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double rs = 0.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const cplx<double> v = p[i * N + j];
      X.a[i][j] = mk(-eps * v.im, eps * v.re);
      rs += sqrt(v.re * v.re + v.im * v.im);
    }
    nrm = rs > nrm ? rs : nrm;
  }
  nrm *= fabs(eps);
  int sq = 0;
  while (nrm > 0.25 && sq < 40) {
    nrm *= 0.5;
    ++sq;
  }
  const double sc = ldexp(1.0, -sq);
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) X.a[i][j] = sc * X.a[i][j];
  Mat<N> E;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) E.a[i][j] = mk(i == j ? 1.0 : 0.0, 0.0);
  for (int k = 16; k >= 1; --k) {   // Horner: E = I + X E / k
    Mat<N> T = mul<N>(X, E);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) E.a[i][j] = (1.0 / k) * T.a[i][j] + mk(i == j ? 1.0 : 0.0, 0.0);
  }
  for (int q = 0; q < sq; ++q) E = mul<N>(E, E);
  cplx<double> *u = U + gid * N * N;
  const Mat<N> Un = mul<N>(E, ld_mat<N>(u, false));
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) u[i * N + j] = Un.a[i][j];
}

// Block partial sums of sum_links tr(pi^2) = sum |pi_ij|^2 (pi Hermitian): a
// block sums the entries of its 256 links, consecutive threads on consecutive
// entries (SU(3) 24^4: 201 us with a thread per link, 33 us).
__global__ __launch_bounds__(256) void k_kinetic_partial(const cplx<double> *__restrict__ pi, double *partial,
                                                         size_t nlinks, int n2) {
  __shared__ double sh[4];
  const size_t l0 = (size_t)blockIdx.x * 256;
  const size_t end = (nlinks - l0 < 256 ? nlinks - l0 : 256) * n2;
  const cplx<double> *p = pi + l0 * n2;
  double s = 0.0;
  for (size_t e = threadIdx.x; e < end; e += 256) {
    const cplx<double> v = p[e];
    s += v.re * v.re + v.im * v.im;
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// pi = sum_a w^a T^a (generators of wd_rep.h's basis: off-diagonal pairs
// (symmetric, antisymmetric) in lexicographic order, then the diagonals).
template <int N>
__global__ __launch_bounds__(256) void k_algebra(cplx<double> *pi, const double *__restrict__ w, size_t nlinks) {
  const size_t l = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= nlinks) return;
  constexpr int NA = N * N - 1;
  const double *wl = w + l * NA;
  cplx<double> m[N][N];
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) m[i][j] = mk(0.0, 0.0);
  int a = 0;
  for (int j = 0; j < N; ++j)
    for (int k = j + 1; k < N; ++k) {
      // (E_jk + E_kj)/2 and (-i E_jk + i E_kj)/2
      const double s = 0.5 * wl[a], t = 0.5 * wl[a + 1];
      m[j][k] = mk(s, -t);
      m[k][j] = mk(s, t);
      a += 2;
    }
  for (int kk = 1; kk < N; ++kk) {
    const double c = wl[a++] / sqrt(2.0 * kk * (kk + 1));
    for (int i = 0; i < kk; ++i) m[i][i].re += c;
    m[kk][kk].re -= kk * c;
  }
  cplx<double> *o = pi + l * N * N;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) o[i * N + j] = m[i][j];
}

// ------------------------------------------------------------------ launch
template <int N>
static hipError_t gf_launch(const void *U, void *F, const Geom &g, double beta, double scale, int accumulate,
                            hipStream_t st) {
  const size_t n = 4 * ((2 * (size_t)g.Vh + 63) / 64);   // (64 sites, direction)
  hipLaunchKernelGGL(k_gauge_force<N>, dim3((unsigned)n), dim3(64), 0, st,
                     (const cplx<double> *)U, (cplx<double> *)F, g, beta, scale, accumulate);
  return hipGetLastError();
}

hipError_t launch_gauge_force(const void *U, void *F, const Geom &g, int N, double beta, double scale,
                              int accumulate, hipStream_t st) {
  switch (N) {
    case 2: return gf_launch<2>(U, F, g, beta, scale, accumulate, st);
    case 3: return gf_launch<3>(U, F, g, beta, scale, accumulate, st);
    case 4: return gf_launch<4>(U, F, g, beta, scale, accumulate, st);
  }
  return hipErrorInvalidValue;
}

// (at most kinetic_blocks, which sizes the workspace)
int plaquette_blocks(const Geom &g) { return (int)((2 * (size_t)g.Vh + 63) / 64); }

hipError_t launch_plaquette_partial(const void *U, double *partial, const Geom &g, int N, hipStream_t st) {
  const dim3 grid(plaquette_blocks(g));
  switch (N) {
    case 2: hipLaunchKernelGGL(k_plaquette_partial<2>, grid, dim3(192), 0, st, (const cplx<double> *)U, partial, g);
      return hipGetLastError();
    case 3: hipLaunchKernelGGL(k_plaquette_partial<3>, grid, dim3(192), 0, st, (const cplx<double> *)U, partial, g);
      return hipGetLastError();
    case 4: hipLaunchKernelGGL(k_plaquette_partial<4>, grid, dim3(192), 0, st, (const cplx<double> *)U, partial, g);
      return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

hipError_t launch_link_update(void *U, const void *pi, const Geom &g, int N, double eps, hipStream_t st) {
  const size_t n = 8 * (size_t)g.Vh;
  const dim3 grid((unsigned)((n + 255) / 256));
  switch (N) {
    case 2: hipLaunchKernelGGL(k_link_update<2>, grid, dim3(256), 0, st, (cplx<double> *)U, (const cplx<double> *)pi,
                               g, eps);
      return hipGetLastError();
    case 3: hipLaunchKernelGGL(k_link_update<3>, grid, dim3(256), 0, st, (cplx<double> *)U, (const cplx<double> *)pi,
                               g, eps);
      return hipGetLastError();
    case 4: hipLaunchKernelGGL(k_link_update<4>, grid, dim3(256), 0, st, (cplx<double> *)U, (const cplx<double> *)pi,
                               g, eps);
      return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

int kinetic_blocks(const Geom &g) { return (int)((8 * (size_t)g.Vh + 255) / 256); }

hipError_t launch_kinetic_partial(const void *pi, double *partial, const Geom &g, int N, hipStream_t st) {
  const size_t nl = 8 * (size_t)g.Vh;
  hipLaunchKernelGGL(k_kinetic_partial, dim3(kinetic_blocks(g)), dim3(256), 0, st, (const cplx<double> *)pi, partial,
                     nl, N * N);
  return hipGetLastError();
}

hipError_t launch_algebra(void *pi, const double *w, const Geom &g, int N, hipStream_t st) {
  const size_t nl = 8 * (size_t)g.Vh;
  const dim3 grid((unsigned)((nl + 255) / 256));
  switch (N) {
    case 2: hipLaunchKernelGGL(k_algebra<2>, grid, dim3(256), 0, st, (cplx<double> *)pi, w, nl);
      return hipGetLastError();
    case 3: hipLaunchKernelGGL(k_algebra<3>, grid, dim3(256), 0, st, (cplx<double> *)pi, w, nl);
      return hipGetLastError();
    case 4: hipLaunchKernelGGL(k_algebra<4>, grid, dim3(256), 0, st, (cplx<double> *)pi, w, nl);
      return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

}  // namespace wd
