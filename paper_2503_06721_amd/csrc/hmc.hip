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
#include "wd_links.h"

namespace wd {

// F = scale * (beta/N) (B - tr B/N)/2 (+ F) per link.  A block takes 16
// consecutive sites; thread = column c (one per wavefront), direction mu, site.
// The links that the staples of the tile have in common go through LDS (44 a
// site, where the staples have 72), in three phases: the sites x-nu, whose
// products with a column stay in registers, the corners x+mu-nu that close the
// lower staples, and x with x+nu.  SU(3) 24^4: 493 us with a lane reading its
// own links; 404 us with a direction of 64 sites per wavefront and each staple's
// three links staged, 6.6 GB through L2 at 16 TB/s, half of every line unused;
// 355 us from this tile with a thread per link, 2.8 GB but four wavefronts a
// CU; 282 us.
template <int N, bool DIRECT>
__global__ __launch_bounds__(64 * N) void k_gauge_force(const cplx<double> *__restrict__ U, cplx<double> *F, Geom g,
                                                        double beta, double scale, int accumulate) {
  using LT = LinkTile<N, 16, 64 * N, DIRECT>;
  constexpr int E = N * N;
  __shared__ cplx<double> buf[LT::elems(16)];
  __shared__ unsigned tab[(16 + 12 + 16) * 16];
  const unsigned b = xcd_range(blockIdx.x, gridDim.x);
  const int c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int mu = (int)(threadIdx.x >> 4) & 3, s = (int)(threadIdx.x & 15);
  // slots: 4 nu + a: U_a(x-nu) | 3 mu + j: U_nu(x+mu-nu), nu the j-th other than mu
  // | a: U_a(x), 4 + 3 b + j: U_a(x+b), a the j-th other than b
  unsigned *t0 = tab, *t1 = tab + 16 * 16, *t2 = tab + 28 * 16;
  if (c == 0) {
    const Site x(g, b * 16 + s);
    const unsigned xp = x.lex + x.shift(g, mu, 1), xm = x.lex + x.shift(g, mu, -1);
    t2[mu * 16 + s] = x.lex * 4 + mu;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int nu = j + (j >= mu);
      t1[(3 * mu + j) * 16 + s] = (xp + x.shift(g, nu, -1)) * 4 + nu;
      t2[(4 + 3 * mu + j) * 16 + s] = xp * 4 + nu;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) t0[(4 * mu + a) * 16 + s] = xm * 4 + a;
  }
  __syncthreads();
  LT::template fetch<16>(buf, U, t0);
  wait_fetch();
  __syncthreads();
  // lower staples U_nu(x+mu-nu)^+ U_mu(x-nu)^+ U_nu(x-nu)
  Vec<N> v[3], A;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int nu = j + (j >= mu);
    v[j] = mulv_dag<N>(LT::at(buf, 4 * nu + mu, s), col<N>(LT::at(buf, 4 * nu + nu, s), c));
  }
  __syncthreads();
  LT::template fetch<12>(buf, U, t1);
  wait_fetch();
  __syncthreads();
  A = mulv_dag<N>(LT::at(buf, 3 * mu, s), v[0]);
  add<N>(A, mulv_dag<N>(LT::at(buf, 3 * mu + 1, s), v[1]));
  add<N>(A, mulv_dag<N>(LT::at(buf, 3 * mu + 2, s), v[2]));
  __syncthreads();
  LT::template fetch<16>(buf, U, t2);
  wait_fetch();
  __syncthreads();
  // upper staples U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int nu = j + (j >= mu);
    add<N>(A, mulv<N>(LT::at(buf, 4 + 3 * mu + j, s),
                      mulv_dag<N>(LT::at(buf, 4 + 3 * nu + mu - (mu > nu), s), col_dag<N>(LT::at(buf, nu, s), c))));
  }
  const Vec<N> M = mulv<N>(LT::at(buf, mu, s), A);
  __syncthreads();
  // column c of M to LDS, row (s, mu) of ROW entries
#pragma unroll
  for (int i = 0; i < N; ++i) buf[(s * 4 + mu) * LT::ROW + i * N + c] = M.a[i];
  __syncthreads();
  // B = (M - M^+)/(2i): B_ij = (M_ij - conj(M_ji)) / (2i)
  const double w = scale * beta / N * 0.5;
  cplx<double> *out = F + (size_t)b * 64 * E;
#pragma unroll
  for (int f = threadIdx.x; f < 64 * E; f += 64 * N) {
    const int m = f / E, e = f - m * E, i = e / N, j = e - i * N;
    const cplx<double> *r = buf + m * LT::ROW;
    const double re = r[i * N + j].re - r[j * N + i].re, im = r[i * N + j].im + r[j * N + i].im;
    double trB = 0.0;
    if (i == j)
#pragma unroll
      for (int k = 0; k < N; ++k) trB += r[k * N + k].im;
    cplx<double> o = mk(w * (0.5 * im - trB / N), w * (-0.5 * re));
    if (accumulate) o = o + out[f];
    out[f] = o;
  }
}

// Sum over the sites of Re tr P_mu,nu / N over the six planes; a partial sum
// per block of 64 sites, which it takes in two tiles of 32, a thread per (plane,
// site).  tr P = sum_ij a_ij conj(b_ij), a = U_mu(x) U_nu(x+mu), b = U_nu(x)
// U_mu(x+nu), the 16 links of a site staged once for its planes.  SU(3) 24^4:
// 336 us with a lane reading its own links, 116 us with each plane's staged on
// their own (24 a site), 107 us (with a thread per column, as above, 170: a
// product of two reads each column's factor again).
template <int N, bool DIRECT>
__global__ __launch_bounds__(192) void k_plaquette_partial(const cplx<double> *__restrict__ U, double *partial,
                                                           Geom g) {
  constexpr int S = 32;
  using LT = LinkTile<N, S, 192, DIRECT>;
  __shared__ cplx<double> buf[LT::elems(16)];
  __shared__ unsigned tab[16 * S];
  __shared__ double sh[3];
  const unsigned V = 2 * (unsigned)g.Vh;
  const unsigned blk = xcd_range(blockIdx.x, gridDim.x);
  const int p = (int)(threadIdx.x >> 5), s = (int)(threadIdx.x & 31);   // (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
  const int mu = p < 3 ? 0 : p < 5 ? 1 : 2, nu = p < 3 ? p + 1 : p < 5 ? p - 1 : 3;
  double sum = 0.0;
#pragma unroll 1
  for (int q = 0; q < 2; ++q) {
    const unsigned lex = blk * 64 + q * S + s;
    const Site x(g, lex < V ? lex : V - 1);
    if (p < 4) {   // slots a: U_a(x), 4 + 3 b + j: U_a(x+b), a the j-th other than b
      const unsigned xp = x.lex + x.shift(g, p, 1);
      tab[p * S + s] = x.lex * 4 + p;
#pragma unroll
      for (int j = 0; j < 3; ++j) tab[(4 + 3 * p + j) * S + s] = xp * 4 + j + (j >= p);
    }
    __syncthreads();
    LT::template fetch<16>(buf, U, tab);
    wait_fetch();
    __syncthreads();
    const Mat<N> a = mul<N>(ld_mat<N>(LT::at(buf, mu, s), false),
                            ld_mat<N>(LT::at(buf, 4 + 3 * mu + nu - (nu > mu), s), false));
    const unsigned i = after<N>(s, a);
    const Mat<N> b = mul<N>(ld_mat<N>(LT::at(buf, nu, i), false),
                            ld_mat<N>(LT::at(buf, 4 + 3 * nu + mu - (mu > nu), i), false));
    double tr = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        tr = fma(a.a[k][j].re, b.a[k][j].re, tr);
        tr = fma(a.a[k][j].im, b.a[k][j].im, tr);
      }
    if (lex < V) sum += tr / N;
    __syncthreads();
  }
  sum = block_sum(sum, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = sum;
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
  const size_t n = g.Vh / 8;   // 16 sites (every extent is even)
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(64 * N), 0, st, (const cplx<double> *)U, (cplx<double> *)F, g,
                       beta, scale, accumulate);
    return hipGetLastError();
  };
  return direct_ok(U) ? go(k_gauge_force<N, true>) : go(k_gauge_force<N, false>);
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

template <int N>
static hipError_t plaq_launch(const void *U, double *partial, const Geom &g, hipStream_t st) {
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(plaquette_blocks(g)), dim3(192), 0, st, (const cplx<double> *)U, partial, g);
    return hipGetLastError();
  };
  return direct_ok(U) ? go(k_plaquette_partial<N, true>) : go(k_plaquette_partial<N, false>);
}

hipError_t launch_plaquette_partial(const void *U, double *partial, const Geom &g, int N, hipStream_t st) {
  switch (N) {
    case 2: return plaq_launch<2>(U, partial, g, st);
    case 3: return plaq_launch<3>(U, partial, g, st);
    case 4: return plaq_launch<4>(U, partial, g, st);
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
