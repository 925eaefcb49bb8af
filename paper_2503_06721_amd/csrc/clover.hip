// Clover improvement (Sec. 6.1.2; exponential form Sec. 6.1.3): the site-diagonal blocks
//   D_ee + D_oo = (4 + m) + c_sw (i/4) sum_{mu,nu} sigma_mu,nu F_mu,nu
// (or, exponential form, (4 + m) exp(c_sw/(4+m) (i/4) sum sigma F)), with
// F_mu,nu = (Q_mu,nu - Q_mu,nu^+)/8 and Q the sum of the four clover leaves of
// the (mu, nu) plane at x, all starting at x and turning from mu to nu.
//
// The leaves are products of fundamental links (N x N); each leaf is mapped to
// the fermion representation entry by entry (wd_rep.h), which is far cheaper
// than multiplying d_R x d_R represented links.  Since R(L)^+ = R(L^+),
//   F_R = sum_leaves (R(L) - R(L)^+) / 8.
// sigma_mu,nu = (i/2)[gamma_mu, gamma_nu] commutes with gamma_5 =
// diag(1,1,-1,-1), so each site holds two 2d x 2d chirality blocks (spins
// {0,1} and {2,3}).  Stored per parity: the even sites keep the blocks
// (D_ee), the odd sites their inverses (D_oo^{-1}), which is what the
// even-odd operator D-hat = D_ee - D_eo D_oo^{-1} D_oe applies.  All these
// blocks are Hermitian, so only the upper triangle (row-major, diagonal
// included: 2d(2d+1)/2 complex entries) is stored.
#include "wd_common.h"
#include "wd_kernels.h"
#include "wd_rep.h"

namespace wd {

// Plane p = 0..5 <-> (mu, nu) = (0,1) (0,2) (0,3) (1,2) (1,3) (2,3).
__device__ __forceinline__ void plane_dirs(int p, int &mu, int &nu) {
  mu = p < 3 ? 0 : p < 5 ? 1 : 2;
  nu = p < 3 ? p + 1 : p < 5 ? p - 1 : 3;
}

// Position of entry (i, j), i <= j, of the packed upper triangle of an
// NB x NB Hermitian block; entry (j, i) is its conjugate.
__host__ __device__ constexpr int tri_index(int NB, int i, int j) { return i * NB - i * (i - 1) / 2 + (j - i); }

// Hermitian n x n matrices as n^2 reals: the diagonal, then Re and Im of the
// entries (i, j), i < j; position of that pair's real part.
__host__ __device__ constexpr int herm_pair(int n, int i, int j) {
  return n + 2 * (i * n - i * (i + 1) / 2 + (j - i - 1));
}

// Entry (i, j) of a packed Hermitian block (any i, j).
template <typename T>
__device__ __forceinline__ cplx<T> herm_entry(const cplx<T> *P, size_t es, int NB, int i, int j) {
  if (i <= j) return P[(size_t)tri_index(NB, i, j) * es];
  const cplx<T> v = P[(size_t)tri_index(NB, j, i) * es];
  return mk<T>(v.re, -v.im);
}

// Workgroups are dispatched to the 8 XCDs round-robin; block b is given the
// logical index that makes each XCD's blocks one contiguous range, so that
// consecutive logical blocks (the planes or directions of one site chunk)
// run on the same XCD and share its L2 (the leaf and gather kernels; the F
// kernel is faster without it).
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned n) {
  const unsigned q = n >> 3, rmd = n & 7, x = b & 7, j = b >> 3;
  return x * q + (x < rmd ? x : rmd) + j;
}

// Sites c + a e_lo + b e_hi (|a|, |b| <= 1) around one site in the plane
// (lo, hi), lexicographic: only the two coordinates that move are wrapped,
// by compare and select (no integer division).  Site indices are 32-bit (a
// lattice has at most 2^30 sites).
struct PlaneNb {
  int base, slo, shi, clo, chi, Llo, Lhi;
  __device__ __forceinline__ static int pick(int i, int v0, int v1, int v2, int v3) {
    return i == 0 ? v0 : i == 1 ? v1 : i == 2 ? v2 : v3;
  }
  __device__ __forceinline__ PlaneNb(const Geom &g, const int (&c)[4], unsigned lex, int lo, int hi) {
    const int sz = g.Z, sy = g.Y * g.Z, sx = sy * g.X;
    base = (int)lex;
    slo = pick(lo, sx, sy, sz, 1);
    shi = pick(hi, sx, sy, sz, 1);
    clo = pick(lo, c[0], c[1], c[2], c[3]);
    chi = pick(hi, c[0], c[1], c[2], c[3]);
    Llo = pick(lo, g.T, g.X, g.Y, g.Z);
    Lhi = pick(hi, g.T, g.X, g.Y, g.Z);
  }
  __device__ __forceinline__ unsigned at(int a, int b) const {
    const int qa = clo + a, qb = chi + b;
    const int da = qa < 0 ? a + Llo : qa >= Llo ? a - Llo : a;
    const int db = qb < 0 ? b + Lhi : qb >= Lhi ? b - Lhi : b;
    return (unsigned)(base + da * slo + db * shi);
  }
};
// Coordinates of lexicographic site lex.
__device__ __forceinline__ void lex_coords(const Geom &g, unsigned lex, int (&c)[4]) {
  unsigned r = lex;
  c[3] = (int)(r % (unsigned)g.Z); r /= (unsigned)g.Z;
  c[2] = (int)(r % (unsigned)g.Y); r /= (unsigned)g.Y;
  c[1] = (int)(r % (unsigned)g.X);
  c[0] = (int)(r / (unsigned)g.X);
}

// The clover kernels read the fundamental links from a structure-of-arrays
// copy Us[mu][N*N][V] (lexicographic site minor; k_links_soa), so that the
// lanes of a wavefront, on consecutive sites, read consecutive addresses.  The
// direction (and plane) is the same for all lanes of a wavefront, so each
// entry row has a scalar base address and a lane one 32-bit byte offset, which
// reaches kNarrowSites sites of 16 bytes.  Of the calls whose fields and scratch
// a 288 GB card can hold, only the SU(2) fundamental clover field (1056 bytes a
// site with FP32 blocks, up to 2.9e8 sites) goes beyond: F_launch gives it 64-bit
// offsets there.  (The next is SU(2) d_R = 3 at 1712 bytes; a force takes 3136 or
// more.)
constexpr size_t kNarrowSites = (size_t)1 << 28;
template <typename V>
__device__ __forceinline__ const V *at(const V *base, size_t off) {
  return base + off;
}
template <typename V>
__device__ __forceinline__ V *at(V *base, size_t off) {
  return base + off;
}

template <int N, typename Off>
__device__ __forceinline__ void load_link(cplx<double> (&u)[N][N], const cplx<double> *Us, size_t V, Off lex, int mu,
                                          bool dag) {
  const cplx<double> *p = Us + (size_t)__builtin_amdgcn_readfirstlane(mu) * N * N * V;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const cplx<double> v = *at(p + (size_t)(dag ? j * N + i : i * N + j) * V, lex);
      u[i][j] = dag ? mk(v.re, -v.im) : v;
    }
}

// Us[mu][e][lex] = U[lex][mu][e] (canonical [T][X][Y][Z][4][N][N] complex).
// A block transposes 64 sites through LDS: the 64 x 4 N^2 entries are read in
// canonical order (consecutive threads, consecutive addresses) and written
// per (mu, e) as a run of 64 consecutive sites.
template <int N>
__global__ __launch_bounds__(256) void k_links_soa(const cplx<double> *__restrict__ U, cplx<double> *__restrict__ Us,
                                                   size_t V) {
  constexpr int E = 4 * N * N;   // complex entries per site
  constexpr int S = E + 1;       // LDS row, padded against bank conflicts
  __shared__ cplx<double> t[64 * S];
  const size_t s0 = (size_t)blockIdx.x * 64;
  const int ns = V - s0 < 64 ? (int)(V - s0) : 64;
  const cplx<double> *src = U + s0 * E;
  for (int k = threadIdx.x; k < ns * E; k += 256) t[(k / E) * S + k % E] = src[k];
  __syncthreads();
  for (int k = threadIdx.x; k < 64 * E; k += 256) {
    const int j = k >> 6, site = k & 63;   // j = mu N^2 + e
    if (site < ns) Us[(size_t)j * V + s0 + site] = t[site * S + j];
  }
}

template <int N>
static hipError_t links_soa_launch(const void *U, double *Us, const Geom &g, hipStream_t st) {
  const size_t V = 2 * (size_t)g.Vh;
  hipLaunchKernelGGL((k_links_soa<N>), dim3((unsigned)((V + 63) / 64)), dim3(256), 0, st,
                     (const cplx<double> *)U, (cplx<double> *)Us, V);
  return hipGetLastError();
}

// acc = acc * u
template <int N>
__device__ __forceinline__ void mul_right(cplx<double> (&acc)[N][N], const cplx<double> (&u)[N][N]) {
  cplx<double> r[N][N];
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      cplx<double> s = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < N; ++k) s = cfma(acc[i][k], u[k][j], s);
      r[i][j] = s;
    }
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) acc[i][j] = r[i][j];
}

// Leaf k of plane (mu, nu) at x as four (site offset (a_mu, b_nu), direction,
// dagger) factors.
struct LeafStep {
  signed char a, b, dir, dag;   // dir 0 = mu, 1 = nu
};
// Used in loops unrolled over (leaf, step), so that every lookup folds into a
// constant.
__device__ constexpr LeafStep kLeafC[4][4] = {
    // U_mu(x) U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
    {{0, 0, 0, 0}, {1, 0, 1, 0}, {0, 1, 0, 1}, {0, 0, 1, 1}},
    // U_nu(x) U_mu(x-mu+nu)^+ U_nu(x-mu)^+ U_mu(x-mu)
    {{0, 0, 1, 0}, {-1, 1, 0, 1}, {-1, 0, 1, 1}, {-1, 0, 0, 0}},
    // U_mu(x-mu)^+ U_nu(x-mu-nu)^+ U_mu(x-mu-nu) U_nu(x-nu)
    {{-1, 0, 0, 1}, {-1, -1, 1, 1}, {-1, -1, 0, 0}, {0, -1, 1, 0}},
    // U_nu(x-nu)^+ U_mu(x-nu) U_nu(x-nu+mu) U_mu(x)^+
    {{0, -1, 1, 1}, {0, -1, 0, 0}, {1, -1, 1, 0}, {0, 0, 0, 1}},
};

// F scratch: F[p][A][B] of every site, [6][D][D][V] complex FP64.  Thread per
// (plane, site), consecutive threads on consecutive sites.  Off: type of the
// lanes' site offsets (load_link).
template <int N, int REP, typename Off>
__global__ __launch_bounds__(256) void k_clover_F(const cplx<double> *__restrict__ U, cplx<double> *__restrict__ F,
                                                  Geom g) {
  constexpr int D = rep_dim(N, REP);
  const size_t V = 2 * (size_t)g.Vh;
  const unsigned gid = blockIdx.x * 256u + threadIdx.x;   // below 6 V, V < 2^29
  // 64-site chunks, the six planes of a chunk in consecutive wavefronts (the
  // planes that share a link direction read it close together in time)
  const unsigned chunk = gid / 384u;
  const int r6 = (int)(gid - chunk * 384u);
  const int p = __builtin_amdgcn_readfirstlane(r6 >> 6);
  const unsigned lex = chunk * 64u + (r6 & 63);
  if (lex >= V) return;
  int mu, nu;
  plane_dirs(p, mu, nu);
  int c[4];
  lex_coords(g, lex, c);
  const PlaneNb pn(g, c, lex, mu, nu);
  cplx<double> *Fp = F + (size_t)p * D * D * V;
  if constexpr (REP == 0) {
    // fundamental representation (R = 1): the four leaves summed in
    // registers, F = (Q - Q^+)/8 written once (the other representations
    // accumulate (R(L) - R(L)^+)/8 leaf by leaf in F below: their d_R^2
    // accumulators do not fit in registers beside the leaf products)
    constexpr bool FUND = true;
    constexpr int DA = FUND ? N : D;
    cplx<double> acc[DA][DA];
#pragma unroll
    for (int A = 0; A < DA; ++A)
#pragma unroll
      for (int B = 0; B < DA; ++B) acc[A][B] = mk(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cplx<double> L[N][N];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const LeafStep st = kLeafC[k][f];
        cplx<double> u[N][N];
        load_link<N>(u, U, V, (Off)pn.at(st.a, st.b), st.dir ? nu : mu, st.dag != 0);
        if (f == 0) {
#pragma unroll
          for (int i = 0; i < N; ++i)
#pragma unroll
            for (int j = 0; j < N; ++j) L[i][j] = u[i][j];
        } else {
          mul_right<N>(L, u);
        }
      }
#pragma unroll
      for (int A = 0; A < DA; ++A)
#pragma unroll
        for (int B = 0; B < DA; ++B) {
          if constexpr (FUND) {
            acc[A][B] = acc[A][B] + L[A][B];
          } else {
            const cplx<double> rab = rep_entry<N, REP>(L, A, B), rba = rep_entry<N, REP>(L, B, A);
            acc[A][B] = acc[A][B] + mk(rab.re - rba.re, rab.im + rba.im);
          }
        }
      // one leaf's links live at a time
      __builtin_amdgcn_sched_barrier(0);
    }
    // F = (Q - Q^+)/8 (fundamental), or the sum of (R(L) - R(L)^+)/8
#pragma unroll
    for (int A = 0; A < DA; ++A)
#pragma unroll
      for (int B = 0; B < DA; ++B) {
        const cplx<double> v = FUND ? mk(0.125 * (acc[A][B].re - acc[B][A].re), 0.125 * (acc[A][B].im + acc[B][A].im))
                                    : 0.125 * acc[A][B];
        *at(Fp + (size_t)(A * D + B) * V, (Off)lex) = v;
      }
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    cplx<double> L[N][N];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const LeafStep s = kLeafC[k][f];
      cplx<double> u[N][N];
      load_link<N>(u, U, V, (Off)pn.at(s.a, s.b), s.dir ? nu : mu, s.dag != 0);
      if (f == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int j = 0; j < N; ++j) L[i][j] = u[i][j];
      } else {
        mul_right<N>(L, u);
      }
    }
    // F += (R(L) - R(L)^+) / 8
    for (int A = 0; A < D; ++A)
      for (int B = 0; B < D; ++B) {
        const cplx<double> rab = rep_entry<N, REP>(L, A, B), rba = rep_entry<N, REP>(L, B, A);
        cplx<double> v = mk(0.125 * (rab.re - rba.re), 0.125 * (rab.im + rba.im));
        cplx<double> *o = at(Fp + (size_t)(A * D + B) * V, (Off)lex);
        if (k > 0) v = v + *o;
        *o = v;
      }
  }
}

// sigma blocks: S.v[p][c][s][t] = 2 x (chirality block c of sigma_mu,nu)_st for
// plane p (the factor 2 counts the (nu, mu) term of the sum).
struct SigmaBlocks {
  cplx<double> v[6][2][2][2];
};

// Hermitian NB x NB matrices in registers: the real diagonal and the upper
// triangle, every index a compile-time constant.
template <int NB>
struct Herm {
  double d[NB];
  cplx<double> o[NB * (NB - 1) / 2];
  static constexpr int at(int i, int j) { return i * (NB - 1) - i * (i - 1) / 2 + (j - i - 1); }   // i < j
  // entry (i, j), i != j
  __device__ __forceinline__ cplx<double> off(int i, int j) const {
    if (i < j) return o[at(i, j)];
    const cplx<double> v = o[at(j, i)];
    return mk(v.re, -v.im);
  }
};

// f a b + g for commuting a, b (the product is then Hermitian: only its
// diagonal and upper triangle are formed), g times the unit matrix.
template <int NB>
__device__ __forceinline__ Herm<NB> herm_mul(const Herm<NB> &a, const Herm<NB> &b, double f, double g) {
  Herm<NB> r;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    double s = a.d[i] * b.d[i];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      if (k == i) continue;
      const cplx<double> x = a.off(i, k), y = b.off(i, k);   // b_ki = conj(b_ik)
      s = fma(x.re, y.re, s);
      s = fma(x.im, y.im, s);
    }
    r.d[i] = fma(f, s, g);
#pragma unroll
    for (int j = i + 1; j < NB; ++j) {
      const cplx<double> aij = a.off(i, j), bij = b.off(i, j);
      cplx<double> t = mk(a.d[i] * bij.re, a.d[i] * bij.im);
      t.re = fma(b.d[j], aij.re, t.re);
      t.im = fma(b.d[j], aij.im, t.im);
#pragma unroll
      for (int k = 0; k < NB; ++k)
        if (k != i && k != j) t = cfma(a.off(i, k), b.off(k, j), t);
      r.o[Herm<NB>::at(i, j)] = mk(f * t.re, f * t.im);
    }
  }
  return r;
}

// Scaling 2^-sq that brings the norm nrm below 1/4, where the Taylor series of
// degree kTaylor gives exp: the first dropped term is below 0.25^13 / 13! ~ 2e-18.
constexpr int kTaylor = 12;
__device__ __forceinline__ int exp_squarings(double nrm) {
  int sq = 0;
  while (nrm > 0.25 && sq < 60) {
    nrm *= 0.5;
    ++sq;
  }
  return sq;
}

// Exponential form, d_R <= 3: thread per (site, chirality block), the block
// index fastest as in k_clover_finish_reg.  Everything is a polynomial in the
// Hermitian A = C / (4 + m) (odd sites: -A), so a product costs its upper
// triangle (432 FMA for d_R = 3 instead of 864) and three matrices stay in
// registers (two waves per SIMD): bound by FP64 arithmetic.  SU(3) FUND 32^4:
// 3604 us with general matrices, which spilled to scratch; 575 us.
template <int D, typename T>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_clover_finish_exp(
    const cplx<double> *__restrict__ F, void *__restrict__ clov, Geom g, SigmaBlocks S, double m0, double csw) {
  constexpr int NB = 2 * D;
  const size_t V = 2 * (size_t)g.Vh;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= 2 * V) return;
  const int c = (int)(gid & 1);
  const unsigned lex = (unsigned)(gid >> 1);
  unsigned r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  const double m4 = 4.0 + m0;
  // A = f sum_p (i S_p) F_p, f = c_sw / (4 (4 + m)); i S_p and F_p are
  // anti-Hermitian and Hermitian-times-i, their products' sum Hermitian
  const double f = (par == 0 ? 0.25 : -0.25) * csw / m4;
  Herm<NB> A;
#pragma unroll
  for (int i = 0; i < NB; ++i) A.d[i] = 0.0;
#pragma unroll
  for (int k = 0; k < NB * (NB - 1) / 2; ++k) A.o[k] = mk(0.0, 0.0);
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    cplx<double> fp[D][D];
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
      for (int b = 0; b < D; ++b) fp[a][b] = F[((size_t)p * D * D + a * D + b) * V + lex];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int tt = s2; tt < 2; ++tt) {
        const cplx<double> sv = S.v[p][c][s2][tt];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
          for (int b = 0; b < D; ++b) {
            const int i = s2 * D + a, j = tt * D + b;
            if (i == j) {   // Re(i sv fp) = -Im(sv fp)
              A.d[i] = fma(-sv.re, fp[a][b].im, A.d[i]);
              A.d[i] = fma(-sv.im, fp[a][b].re, A.d[i]);
            } else if (i < j) {
              cplx<double> &o = A.o[Herm<NB>::at(i, j)];
              o = cfma(mk(-sv.im, sv.re), fp[a][b], o);
            }
          }
      }
    // one plane's F entries live at a time
    __builtin_amdgcn_sched_barrier(0);
  }
  // largest column sum of |A| (Hermitian: row sums)
  double nrm = 0.0;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (j == i) s += fabs(A.d[i]);
      else {
        const cplx<double> v = A.off(i, j);
        s += sqrt(v.re * v.re + v.im * v.im);
      }
    }
    nrm = s > nrm ? s : nrm;
  }
  const int sq = exp_squarings(nrm * fabs(f));
  const double sc = ldexp(f, -sq);
#pragma unroll
  for (int i = 0; i < NB; ++i) A.d[i] *= sc;
#pragma unroll
  for (int k = 0; k < NB * (NB - 1) / 2; ++k) A.o[k] = sc * A.o[k];
  // Horner: E = 1 + A (1 + A/2 (1 + A/3 (... (1 + A/K)))), then the squarings
  Herm<NB> E;
#pragma unroll
  for (int i = 0; i < NB; ++i) E.d[i] = fma(1.0 / kTaylor, A.d[i], 1.0);
#pragma unroll
  for (int k = 0; k < NB * (NB - 1) / 2; ++k) E.o[k] = (1.0 / kTaylor) * A.o[k];
#pragma unroll 1
  for (int k = kTaylor - 1; k >= 1; --k) E = herm_mul<NB>(A, E, 1.0 / k, 1.0);
#pragma unroll 1
  for (int q = 0; q < sq; ++q) E = herm_mul<NB>(E, E, 1.0, 0.0);
  // even: (4+m) exp(A); odd: exp(-A)/(4+m)
  const double e = par == 0 ? m4 : 1.0 / m4;
  constexpr int NT = NB * (NB + 1) / 2;
  cplx<T> *dst = static_cast<cplx<T> *>(clov) + ((size_t)(par * 2 + c) * NT) * g.stride + cb;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    dst[(size_t)tri_index(NB, i, i) * g.stride] = mk<T>((T)(e * E.d[i]), (T)0);
#pragma unroll
    for (int j = i + 1; j < NB; ++j) {
      const cplx<double> v = E.off(i, j);
      dst[(size_t)tri_index(NB, i, j) * g.stride] = mk<T>((T)(e * v.re), (T)(e * v.im));
    }
  }
}

// Exchange-method (Gauss-Jordan) inverse with partial pivoting of one NB x NB
// matrix by NB lanes, lane i holding row i in w; every lane of the 64-lane
// block calls it (barriers).  Step k takes the row p_k of largest |w_k| not
// yet taken (a NaN counts as larger than any number, so that every row is taken
// once and the NaN reaches all of the inverse); afterwards lane p_k, whose `mine`
// is k, holds w[j] = (A^-1)[k][p_j].  The columns rotate one place per step, so
// that the step's column is always 0 and w stays in registers.  Returns
// log|det A|.
template <int NB>
__device__ __forceinline__ double rows_exchange(cplx<double> (&w)[NB], cplx<double> (*sh)[NB + 1], int *perm, int i,
                                                bool lane_used, int &mine) {
  bool taken = false;
  double ld = 0.0;
  mine = 0;
#pragma unroll 1
  for (int k = 0; k < NB; ++k) {
    __syncthreads();
    if (lane_used) sh[i][NB] = mk(taken ? -1.0 : w[0].re * w[0].re + w[0].im * w[0].im, 0.0);
    __syncthreads();
    int p = 0;
    double best = -1.0;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const double v = sh[q][NB].re;
      const bool up = v > best || (isnan(v) && !isnan(best));
      p = up ? q : p;
      best = up ? v : best;
    }
    ld += 0.5 * log(best);
    if (i == p) {
      const cplx<double> d = w[0];
      const double dn = 1.0 / (d.re * d.re + d.im * d.im);
      const cplx<double> di = mk(d.re * dn, -d.im * dn);
      w[0] = mk(1.0, 0.0);
#pragma unroll
      for (int j = 0; j < NB; ++j) w[j] = cmul(w[j], di);
      if (lane_used) {
        perm[k] = p;
#pragma unroll
        for (int j = 0; j < NB; ++j) sh[0][j] = w[j];
      }
      taken = true;
      mine = k;
    }
    __syncthreads();
    if (i != p) {
      const cplx<double> f = w[0];
      w[0] = mk(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < NB; ++j) w[j] = w[j] - cmul(f, sh[0][j]);
    }
    const cplx<double> w0 = w[0];
#pragma unroll
    for (int j = 0; j + 1 < NB; ++j) w[j] = w[j + 1];
    w[NB - 1] = w0;
  }
  __syncthreads();
  return ld;
}

// Larger blocks (d_R = 6, and d_R = 4 in the exponential form): NB = 2 d_R
// lanes per (site, chirality block), lane i holding row i and reading other
// rows from LDS; 64-lane blocks of MPB matrices, the lanes past them following
// the barriers.  Exponential form: Horner and squarings as above on general
// rows.  Regular form: D_ee as assembled on even sites, on odd sites its
// inverse (rows_exchange).  (One lane per whole matrix spills it to scratch: SU(3) SYM
// 16^4, the whole field: 5025 us so, 1160 us here, regular; 11244 and 2571 us
// exponential.)
template <int D, typename T>
__global__ __launch_bounds__(64) void k_clover_finish_rows(const cplx<double> *__restrict__ F, void *__restrict__ clov,
                                                           Geom g, SigmaBlocks S, double m0, double csw, int expo) {
  constexpr int NB = 2 * D, MPB = 64 / NB;
  __shared__ cplx<double> sh[MPB][NB][NB + 1];
  const size_t V = 2 * (size_t)g.Vh;
  const int mloc0 = (int)threadIdx.x / NB;
  const bool lane_used = mloc0 < MPB;
  const int mloc = lane_used ? mloc0 : MPB - 1;
  const int i = lane_used ? (int)threadIdx.x - mloc * NB : 0;   // row of this lane
  const size_t m0g = (size_t)blockIdx.x * MPB + mloc;
  const bool valid = lane_used && m0g < 2 * V;
  const size_t mg = m0g < 2 * V ? m0g : 2 * V - 1;
  const int c = (int)(mg / V);
  const unsigned lex = (unsigned)(mg - (size_t)c * V);
  unsigned r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  const int si = i / D, ai = i - si * D;   // row i = (spin si, colour ai)
  const double m4 = 4.0 + m0;
  // row i of (i/4) c_sw sum_p S[p][c][s][t] F_p[a][b]
  cplx<double> a[NB];
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int b = 0; b < D; ++b) {
      cplx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int p = 0; p < 6; ++p)
        acc = cfma(S.v[p][c][si][tt], F[((size_t)p * D * D + ai * D + b) * V + lex], acc);
      a[tt * D + b] = mk(-0.25 * csw * acc.im, 0.25 * csw * acc.re);
    }
  double scale = 1.0;
  if (expo) {   // even: (4+m) exp(a/(4+m)); odd: exp(-a/(4+m))/(4+m)
    double rs = 0.0;   // row sum of |a|: the largest is the norm (Hermitian)
#pragma unroll
    for (int j = 0; j < NB; ++j) rs += sqrt(a[j].re * a[j].re + a[j].im * a[j].im);
    if (lane_used) sh[mloc][i][NB] = mk(rs, 0.0);
    __syncthreads();
    double nrm = 0.0;
    for (int j = 0; j < NB; ++j) nrm = sh[mloc][j][NB].re > nrm ? sh[mloc][j][NB].re : nrm;
    const double f = (par == 0 ? 1.0 : -1.0) / m4;
    const int sq = exp_squarings(nrm * fabs(f));
    int sqmax = sq;   // every lane takes part in every barrier
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const int o = __shfl_xor(sqmax, off, 64);
      sqmax = o > sqmax ? o : sqmax;
    }
    const double sc = ldexp(f, -sq);
    cplx<double> e[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      a[j] = sc * a[j];
      e[j] = mk(i == j ? 1.0 : 0.0, 0.0);
    }
    for (int k = kTaylor; k >= -sqmax + 1; --k) {   // k >= 1: Horner; k <= 0: squarings
      __syncthreads();
      if (lane_used)
#pragma unroll
        for (int j = 0; j < NB; ++j) sh[mloc][i][j] = e[j];
      __syncthreads();
      const bool horner = k >= 1, on = horner || 1 - k <= sq;
      const double rk = horner ? 1.0 / k : 1.0;
      cplx<double> row[NB], n[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) row[q] = mk(horner ? a[q].re : e[q].re, horner ? a[q].im : e[q].im);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        cplx<double> s = mk(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < NB; ++q) s = cfma(row[q], sh[mloc][q][j], s);
        n[j] = mk(fma(rk, s.re, horner && i == j ? 1.0 : 0.0), rk * s.im);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) e[j] = mk(on ? n[j].re : e[j].re, on ? n[j].im : e[j].im);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) a[j] = e[j];
    scale = par == 0 ? m4 : 1.0 / m4;
    __syncthreads();
    if (lane_used)
#pragma unroll
      for (int j = 0; j < NB; ++j) sh[mloc][i][j] = a[j];
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j) a[j].re += i == j ? m4 : 0.0;
    // every matrix goes through the steps (barriers); even sites store a as it is
    cplx<double> w[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) w[j] = a[j];
    __shared__ int perm[MPB][NB];
    int mine;
    rows_exchange<NB>(w, sh[mloc], perm[mloc], i, lane_used, mine);
    if (lane_used)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (par == 0) sh[mloc][i][j] = a[j];
        else sh[mloc][mine][perm[mloc][j]] = w[j];
      }
  }
  __syncthreads();
  if (!valid) return;
  constexpr int NT = NB * (NB + 1) / 2;
  cplx<T> *dst = static_cast<cplx<T> *>(clov) + ((size_t)(par * 2 + c) * NT) * g.stride + cb;
  for (int j = i; j < NB; ++j) {
    // Hermitian up to rounding: store the mean of (i,j) and conj(j,i)
    const cplx<double> u = sh[mloc][i][j], l = sh[mloc][j][i];
    const double re = scale * 0.5 * (u.re + l.re), im = scale * 0.5 * (u.im - l.im);
    dst[(size_t)tri_index(NB, i, j) * g.stride] = mk<T>((T)re, (T)(i == j ? 0.0 : im));
  }
}

// In-place Gauss-Jordan inverse with partial pivoting of the NB x NB matrix
// a, every index a compile-time constant so that the matrix stays in
// registers: the row interchange of a step is a set of selects over the rows
// below the diagonal, and the interchanges are undone at the end as column
// interchanges in reverse order (A^-1 = (P A)^-1 P).
template <int NB>
__device__ __forceinline__ void invert_in_place(cplx<double> (&a)[NB][NB]) {
  int piv[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    int p = k;
    double best = a[k][k].re * a[k][k].re + a[k][k].im * a[k][k].im;
#pragma unroll
    for (int r = k + 1; r < NB; ++r) {
      const double m2 = a[r][k].re * a[r][k].re + a[r][k].im * a[r][k].im;
      p = m2 > best ? r : p;
      best = m2 > best ? m2 : best;
    }
    piv[k] = p;
#pragma unroll
    for (int r = k + 1; r < NB; ++r) {
      const bool sw = p == r;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const cplx<double> tk = a[k][j], tr = a[r][j];
        a[k][j] = sw ? tr : tk;
        a[r][j] = sw ? tk : tr;
      }
    }
    const cplx<double> d = a[k][k];
    const double dn = 1.0 / (d.re * d.re + d.im * d.im);
    const cplx<double> di = mk(d.re * dn, -d.im * dn);
    a[k][k] = mk(1.0, 0.0);
#pragma unroll
    for (int j = 0; j < NB; ++j) a[k][j] = cmul(a[k][j], di);
#pragma unroll
    for (int r = 0; r < NB; ++r) {
      if (r == k) continue;
      const cplx<double> f = a[r][k];
      a[r][k] = mk(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < NB; ++j) a[r][j] = a[r][j] - cmul(f, a[k][j]);
    }
  }
#pragma unroll
  for (int k = NB - 1; k >= 0; --k) {
#pragma unroll
    for (int r = k + 1; r < NB; ++r) {
      const bool sw = piv[k] == r;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const cplx<double> tk = a[i][k], tr = a[i][r];
        a[i][k] = sw ? tr : tk;
        a[i][r] = sw ? tk : tr;
      }
    }
  }
}

// Regular clover (no exponential), d_R <= 4: assemble the block from F, add
// the mass term, invert on odd sites, store in precision T, with the block in
// registers throughout.  Thread per (site, chirality block), the
// block index fastest, so that the two threads of a site read the same F
// entries together (F comes from HBM once).
template <int D, typename T>
__global__ __launch_bounds__(64) void k_clover_finish_reg(const cplx<double> *__restrict__ F, void *__restrict__ clov,
                                                          Geom g, SigmaBlocks S, double m0, double csw) {
  constexpr int NB = 2 * D;
  const size_t V = 2 * (size_t)g.Vh;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= 2 * V) return;
  const int c = (int)(gid & 1);
  const size_t lex = gid >> 1;
  size_t r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  cplx<double> M[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) M[i][j] = mk(0.0, 0.0);
  // (i/4) c_sw sum_p S[p][c][s][t] F_p[a][b], plane by plane
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    cplx<double> fp[D][D];
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
      for (int b = 0; b < D; ++b) fp[a][b] = F[((size_t)p * D * D + a * D + b) * V + lex];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const cplx<double> sv = S.v[p][c][s2][tt];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
          for (int b = 0; b < D; ++b) M[s2 * D + a][tt * D + b] = cfma(sv, fp[a][b], M[s2 * D + a][tt * D + b]);
      }
    // one plane's F entries live at a time
    __builtin_amdgcn_sched_barrier(0);
  }
  const double m4 = 4.0 + m0;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const cplx<double> v = M[i][j];
      M[i][j] = mk(-0.25 * csw * v.im + (i == j ? m4 : 0.0), 0.25 * csw * v.re);   // (i/4) c_sw acc (+ 4 + m)
    }
  if (par == 1) invert_in_place<NB>(M);
  constexpr int NT = NB * (NB + 1) / 2;
  cplx<T> *dst = static_cast<cplx<T> *>(clov) + ((size_t)(par * 2 + c) * NT) * g.stride + cb;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = i; j < NB; ++j) {
      // Hermitian up to rounding: store the mean of (i,j) and conj(j,i)
      const double re = 0.5 * (M[i][j].re + M[j][i].re), im = 0.5 * (M[i][j].im - M[j][i].im);
      dst[(size_t)tri_index(NB, i, j) * g.stride] = mk<T>((T)re, (T)(i == j ? 0.0 : im));
    }
}

// out = M_c in on the sites of `parity` (thread per (site, rhs, block); the
// thread reads its block's spin components before writing them, so out may
// alias in).
template <int D, typename T>
__global__ __launch_bounds__(256) void k_clover_apply(cplx<T> *out, const cplx<T> *in, const cplx<T> *__restrict__ clov,
                                                      Geom g, int parity, int nrhs) {
  constexpr int NB = 2 * D;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int rc = blockIdx.y;   // rhs * 2 + block
  const int rr = rc >> 1, c = rc & 1;
  if (i >= g.Vh || rr >= nrhs) return;
  const size_t rbase = (size_t)rr * 4 * D * g.stride + i;
  cplx<T> v[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) v[k] = in[rbase + (size_t)(2 * c * D + k) * g.stride];
  constexpr int NT = NB * (NB + 1) / 2;
  const cplx<T> *M = clov + ((size_t)(parity * 2 + c) * NT) * g.stride + i;
  cplx<T> w[NB];
#pragma unroll
  for (int a = 0; a < NB; ++a) w[a] = mk<T>(0, 0);
  // each stored entry (a, b), a <= b, serves (a, b) and, conjugated, (b, a)
#pragma unroll
  for (int a = 0; a < NB; ++a) {
    const cplx<T> d = M[(size_t)tri_index(NB, a, a) * g.stride];
    w[a] = cfma(d, v[a], w[a]);
#pragma unroll
    for (int b = a + 1; b < NB; ++b) {
      const cplx<T> m = M[(size_t)tri_index(NB, a, b) * g.stride];
      w[a] = cfma(m, v[b], w[a]);
      w[b] = cfma_conj(m, v[a], w[b]);
    }
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) out[rbase + (size_t)(2 * c * D + k) * g.stride] = w[k];
}

// ------------------------------------------------------------------ launch
template <int N, int REP>
static hipError_t F_launch(const void *U, double *F, const Geom &g, hipStream_t st) {
  const size_t n = 384 * ((2 * (size_t)g.Vh + 63) / 64);   // six planes per 64-site chunk
  const dim3 grid((unsigned)((n + 255) / 256));
  const cplx<double> *u = (const cplx<double> *)U;
  cplx<double> *f = (cplx<double> *)F;
  if constexpr (N == 2 && REP == 0) {
    if (2 * (size_t)g.Vh > kNarrowSites) {
      hipLaunchKernelGGL((k_clover_F<N, REP, size_t>), grid, dim3(256), 0, st, u, f, g);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_clover_F<N, REP, unsigned>), grid, dim3(256), 0, st, u, f, g);
  return hipGetLastError();
}

template <int D, typename T>
static hipError_t finish_launch_t(const double *F, void *clov, const Geom &g, const SigmaBlocks &S, double m0,
                                  double csw, int expo, hipStream_t st) {
  const size_t n = 2 * 2 * (size_t)g.Vh;
  const cplx<double> *f = (const cplx<double> *)F;
  if constexpr (D <= 3) {
    if (expo) {
      hipLaunchKernelGGL((k_clover_finish_exp<D, T>), dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, f, clov, g, S,
                         m0, csw);
      return hipGetLastError();
    }
  }
  if constexpr (D <= 4) {
    if (!expo) {
      hipLaunchKernelGGL((k_clover_finish_reg<D, T>), dim3((unsigned)((n + 63) / 64)), dim3(64), 0, st, f, clov, g, S,
                         m0, csw);
      return hipGetLastError();
    }
  }
  if constexpr (D > 3) {
    constexpr int MPB = 64 / (2 * D);
    hipLaunchKernelGGL((k_clover_finish_rows<D, T>), dim3((unsigned)((n + MPB - 1) / MPB)), dim3(64), 0, st, f, clov, g,
                       S, m0, csw, expo);
  }
  return hipGetLastError();
}

template <int D>
static hipError_t finish_launch(const double *F, void *clov, const Geom &g, const SigmaBlocks &S, double m0,
                                double csw, int expo, int prec, hipStream_t st) {
  return prec == 0 ? finish_launch_t<D, double>(F, clov, g, S, m0, csw, expo, st)
                   : finish_launch_t<D, float>(F, clov, g, S, m0, csw, expo, st);
}

static SigmaBlocks sigma_blocks() {
  // gamma_mu = [[0, e_mu], [e_mu^+, 0]], e_0 = -1, e_k = -i sigma_k (Sec. 2.2);
  // sigma_mu,nu = i gamma_mu gamma_nu (mu != nu) = diag(i e_mu e_nu^+, i e_mu^+ e_nu).
  cplx<double> e[4][2][2];
  const cplx<double> z = mk(0.0, 0.0);
  e[0][0][0] = mk(-1.0, 0.0); e[0][0][1] = z; e[0][1][0] = z; e[0][1][1] = mk(-1.0, 0.0);
  // -i sigma_1, -i sigma_2, -i sigma_3
  e[1][0][0] = z; e[1][0][1] = mk(0.0, -1.0); e[1][1][0] = mk(0.0, -1.0); e[1][1][1] = z;
  e[2][0][0] = z; e[2][0][1] = mk(-1.0, 0.0); e[2][1][0] = mk(1.0, 0.0); e[2][1][1] = z;
  e[3][0][0] = mk(0.0, -1.0); e[3][0][1] = z; e[3][1][0] = z; e[3][1][1] = mk(0.0, 1.0);
  auto hmul = [](cplx<double> a, cplx<double> b) { return mk(a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re); };
  auto conj = [](cplx<double> a) { return mk(a.re, -a.im); };
  SigmaBlocks S{};
  const int pm[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
  for (int p = 0; p < 6; ++p) {
    const int mu = pm[p][0], nu = pm[p][1];
    for (int s = 0; s < 2; ++s)
      for (int t = 0; t < 2; ++t) {
        cplx<double> up = z, lo = z;
        for (int k = 0; k < 2; ++k) {
          const cplx<double> a = hmul(e[mu][s][k], conj(e[nu][t][k]));      // (e_mu e_nu^+)_st
          const cplx<double> b = hmul(conj(e[mu][k][s]), e[nu][k][t]);      // (e_mu^+ e_nu)_st
          up = mk(up.re + a.re, up.im + a.im);
          lo = mk(lo.re + b.re, lo.im + b.im);
        }
        // 2 i (...)
        S.v[p][0][s][t] = mk(-2.0 * up.im, 2.0 * up.re);
        S.v[p][1][s][t] = mk(-2.0 * lo.im, 2.0 * lo.re);
      }
  }
  return S;
}

template <int N>
static hipError_t F_launch_n(const void *U, double *F, const Geom &g, int rep, hipStream_t st) {
  switch (rep) {
    case 0: return F_launch<N, 0>(U, F, g, st);
    case 1: return F_launch<N, 1>(U, F, g, st);
    case 2: return F_launch<N, 2>(U, F, g, st);
    case 3:
      if constexpr (N > 2) return F_launch<N, 3>(U, F, g, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_clover_field(void *clov, const void *U, double *F, double *Us, const Geom &g, int N, int rep, int d,
                               double m0, double csw, int expo, int prec, hipStream_t st) {
  hipError_t e = hipErrorInvalidValue;
  switch (N) {
    case 2: e = links_soa_launch<2>(U, Us, g, st); if (e == hipSuccess) e = F_launch_n<2>(Us, F, g, rep, st); break;
    case 3: e = links_soa_launch<3>(U, Us, g, st); if (e == hipSuccess) e = F_launch_n<3>(Us, F, g, rep, st); break;
    case 4: e = links_soa_launch<4>(U, Us, g, st); if (e == hipSuccess) e = F_launch_n<4>(Us, F, g, rep, st); break;
  }
  if (e != hipSuccess) return e;
  const SigmaBlocks S = sigma_blocks();
  switch (d) {
    case 2: return finish_launch<2>(F, clov, g, S, m0, csw, expo, prec, st);
    case 3: return finish_launch<3>(F, clov, g, S, m0, csw, expo, prec, st);
    case 4: return finish_launch<4>(F, clov, g, S, m0, csw, expo, prec, st);
    case 6: return finish_launch<6>(F, clov, g, S, m0, csw, expo, prec, st);
  }
  return hipErrorInvalidValue;
}

template <int D>
static hipError_t apply_launch(void *out, const void *in, const void *clov, const Geom &g, int parity, int nrhs,
                               int prec, hipStream_t st) {
  const dim3 grid((g.Vh + 255) / 256, 2 * nrhs);
  if (prec == 0)
    hipLaunchKernelGGL((k_clover_apply<D, double>), grid, dim3(256), 0, st, (cplx<double> *)out,
                       (const cplx<double> *)in, (const cplx<double> *)clov, g, parity, nrhs);
  else
    hipLaunchKernelGGL((k_clover_apply<D, float>), grid, dim3(256), 0, st, (cplx<float> *)out,
                       (const cplx<float> *)in, (const cplx<float> *)clov, g, parity, nrhs);
  return hipGetLastError();
}

hipError_t launch_clover_apply(void *out, const void *in, const void *clov, const Geom &g, int d, int parity,
                               int nrhs, int prec, hipStream_t st) {
  switch (d) {
    case 2: return apply_launch<2>(out, in, clov, g, parity, nrhs, prec, st);
    case 3: return apply_launch<3>(out, in, clov, g, parity, nrhs, prec, st);
    case 4: return apply_launch<4>(out, in, clov, g, parity, nrhs, prec, st);
    case 6: return apply_launch<6>(out, in, clov, g, parity, nrhs, prec, st);
  }
  return hipErrorInvalidValue;
}

bool clover_supported(int d) { return d == 2 || d == 3 || d == 4 || d == 6; }

// ------------------------------------------------------------ clover force
// Link derivative of a functional whose variation is
//   -2 Re sum_x tr[dM(x) Omega(x)]      (M: the site-diagonal blocks),
// the form of both clover contributions to the HMC force: the pseudofermion
// action with Omega = X Y^+ (X = (x, D_oo^{-1} D_oe x), Y = (D-hat x,
// D_oo^{-1} D_eo^+ D-hat x)) and S_det = -2 sum_{x odd} log|det D_oo| with
// Omega = D_oo^{-1} on the odd sites.
//
// With C = (i c_sw/2) sum_p sigma_p (x) F_p (p = mu < nu) and dM = dC
// (exponential form: tr[dM Omega] = tr[dC Omega'], Omega' = L(A, Omega), the
// Frechet derivative of exp at A = C/(4+m), which is its own adjoint for the
// trace pairing), the variation is (c_sw/8) sum_x sum_p Im tr[dQ_p K_p] with
//   K_p = Lam_p + Lam_p^+,  (Lam_p)_ba = sum_st (sigma_p)_st Omega'_(t b),(s a).
// A leaf l of Q_p varied from the left, R(l) -> exp(i th^b T^b_R) R(l),
// changes Im tr[R(l) K_p] by th^b Re tr[T^b_R R(l) K_p]; its matrix
// g = sum_b Re tr[T^b_R R(l) K_p] T^b is formed in the fundamental by the
// representation pull-back.  A link U inside the leaf, l = B U rest, moves it
// by the generator B T B^+ (l = B' U^+ rest: by -(B'U^+) T (B'U^+)^+), so the
// link's force receives +-B^+ g B with B the fundamental path from the
// leaf's corner up to (forward) or through (dagger) the link.
//
// Pipeline (one lattice): insertion K per site -> leaf matrices g per (plane,
// site) -> gather over the 24 (leaf, corner) pairs holding each link; in the
// fundamental representation the gather takes K itself (k_clover_gather_fund).
// Scratch: K [6][d^2][V] reals, g [6][4][N^2][V] reals (Hermitian matrices: the
// diagonal, then Re and Im of the upper triangle).
//
// K only needs the Hermitian B = Omega + Omega^+ (exponential form: L(A, .) maps
// Hermitian to Hermitian): with the Hermitian sigma_p,
//   (K_p)_ba = sum_c sum_st (sigma_p)_st (B_c)_(t b),(s a).

// Thread per site (regular clover; the exponential form is k_clover_insert_exp
// or _rows): B = X Y^+ + Y X^+ per chirality block, or (DET)
// 2 cdet D_oo^{-1} on the odd sites and 0 on the even ones.  For each entry
// (b, a), b <= a, the eight entries of B it needs are formed once and summed
// for the six planes.  Bound by memory: SU(3) FUND 24^4 160 us writing both
// chiralities' general matrices, 64 us (DET: 57).
template <int D, bool DET>
__global__ __launch_bounds__(64) void k_clover_insert(const cplx<double> *__restrict__ Xe,
                                                      const cplx<double> *__restrict__ Xo,
                                                      const cplx<double> *__restrict__ Ye,
                                                      const cplx<double> *__restrict__ Yo,
                                                      const cplx<double> *__restrict__ clov, double *__restrict__ K,
                                                      Geom g, SigmaBlocks S, double cdet) {
  constexpr int NB = 2 * D;
  constexpr bool HOLD = !DET && D <= 3;   // the spinors stay in registers
  const size_t V = 2 * (size_t)g.Vh;
  const unsigned lex = blockIdx.x * 64u + threadIdx.x;
  if (lex >= V) return;
  unsigned r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  const cplx<double> *X = par ? Xo : Xe, *Y = par ? Yo : Ye;
  const cplx<double> *Mi = clov + (size_t)2 * (NB * (NB + 1) / 2) * g.stride + cb;   // odd sites
  cplx<double> xv[HOLD ? 2 * NB : 1], yv[HOLD ? 2 * NB : 1];
  if constexpr (HOLD) {
#pragma unroll
    for (int k = 0; k < 2 * NB; ++k) {
      xv[k] = X[(size_t)k * g.stride + cb];
      yv[k] = Y[(size_t)k * g.stride + cb];
    }
  }
  const auto entry = [&](int b, int a) {
    cplx<double> bm[2][2][2];   // [c][s][t]: (B_c)_(t b),(s a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
          if constexpr (DET) {
            const cplx<double> m =
                par ? herm_entry(Mi + (size_t)c * (NB * (NB + 1) / 2) * g.stride, g.stride, NB, tt * D + b, s * D + a)
                    : mk(0.0, 0.0);
            bm[c][s][tt] = (2.0 * cdet) * m;
          } else {
            const int i = (2 * c + tt) * D + b, j = (2 * c + s) * D + a;
            cplx<double> xi, yi, xj, yj;
            if constexpr (HOLD) {
              xi = xv[i]; yi = yv[i]; xj = xv[j]; yj = yv[j];
            } else {
              xi = X[(size_t)i * g.stride + cb]; yi = Y[(size_t)i * g.stride + cb];
              xj = X[(size_t)j * g.stride + cb]; yj = Y[(size_t)j * g.stride + cb];
            }
            // x_i conj(y_j) + y_i conj(x_j)
            bm[c][s][tt] = cfma_conj(xj, yi, cfma_conj(yj, xi, mk(0.0, 0.0)));
          }
        }
    for (int p = 0; p < 6; ++p) {
      cplx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) acc = cfma(S.v[p][c][s][tt], bm[c][s][tt], acc);   // S.v holds 2 sigma
      double *k = K + (size_t)p * D * D * V + lex;
      if (b == a) {
        k[(size_t)b * V] = 0.5 * acc.re;
      } else {
        const int e = herm_pair(D, b, a);
        k[(size_t)e * V] = 0.5 * acc.re;
        k[(size_t)(e + 1) * V] = 0.5 * acc.im;
      }
    }
  };
  if constexpr (HOLD) {
#pragma unroll
    for (int b = 0; b < D; ++b)
#pragma unroll
      for (int a = b; a < D; ++a) entry(b, a);
  } else {
    for (int b = 0; b < D; ++b)
      for (int a = b; a < D; ++a) entry(b, a);
  }
}

// Exponential form, d_R > 3: as k_clover_insert_exp below, with general matrices
// and (e, l) <- (e e, l e + e l).
// NB = 2 d_R lanes per (site, chirality block): lane i holds row i of A,
// Omega and of the iterates and reads the other rows from LDS at each matrix
// product (one lane holding whole NB x NB matrices spills them to scratch).
// 64-lane blocks (one wavefront) hold MPB = 64 / NB matrices; the lanes past MPB * NB and past the last matrix follow the barriers and
// store nothing (the former write no LDS either).  Every barrier is reached
// the same number of times by all lanes: the squarings run to the block's
// largest count, a matrix that needs fewer keeping its iterates.
template <int D>
__global__ __launch_bounds__(64) void k_clover_insert_rows(const cplx<double> *Xe, const cplx<double> *Xo,
                                                           const cplx<double> *Ye, const cplx<double> *Yo,
                                                           const cplx<double> *__restrict__ clov,
                                                           const cplx<double> *__restrict__ F,
                                                           double *__restrict__ K, Geom g, SigmaBlocks S,
                                                           double m0, double csw, double cdet) {
  // both chirality blocks of a site in one 64-lane block: K sums over them
  constexpr int NB = 2 * D, MPB = 64 / NB / 2 * 2;
  __shared__ cplx<double> se[MPB][NB][NB], sl[MPB][NB][NB];
  const size_t V = 2 * (size_t)g.Vh;
  const int mloc0 = (int)threadIdx.x / NB;
  const bool lane_used = mloc0 < MPB;
  const int mloc = lane_used ? mloc0 : MPB - 1;
  const int i = lane_used ? (int)threadIdx.x - mloc * NB : 0;   // row of this lane
  const size_t m0g = (size_t)blockIdx.x * MPB + mloc;
  const bool valid = lane_used && m0g < 2 * V;
  const size_t mg = m0g < 2 * V ? m0g : 2 * V - 2 + (m0g & 1);
  const int c = (int)(mg & 1);
  const unsigned lex = (unsigned)(mg >> 1);
  unsigned r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  const int si = i / D, ai = i - si * D;   // row i = (spin si, colour ai) of the block
  cplx<double> om[NB], a[NB];   // row i of B and A
#pragma unroll
  for (int j = 0; j < NB; ++j) om[j] = mk(0.0, 0.0);
  if (Xe) {
    const cplx<double> *X = par ? Xo : Xe, *Y = par ? Yo : Ye;
    const size_t oi = (size_t)((2 * c + si) * D + ai) * g.stride + cb;
    const cplx<double> xi = X[oi], yi = Y[oi];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int sj = j / D, aj = j - sj * D;
      const size_t oj = (size_t)((2 * c + sj) * D + aj) * g.stride + cb;
      om[j] = cfma_conj(X[oj], yi, cfma_conj(Y[oj], xi, om[j]));
    }
  }
  if (cdet != 0.0 && par == 1) {
    const cplx<double> *Mi = clov + (size_t)(2 + c) * (NB * (NB + 1) / 2) * g.stride + cb;
#pragma unroll
    for (int j = 0; j < NB; ++j) om[j] = om[j] + (2.0 * cdet) * herm_entry(Mi, g.stride, NB, i, j);
  }
  // row i of A = (i/4) c_sw sum_p S[p][c][s][t] F_p[a][b] / (4 + m)
  const double f = 0.25 * csw / (4.0 + m0);
#pragma unroll
  for (int tt = 0; tt < 2; ++tt)
#pragma unroll
    for (int b = 0; b < D; ++b) {
      cplx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int p = 0; p < 6; ++p)
        acc = cfma(S.v[p][c][si][tt], F[((size_t)p * D * D + ai * D + b) * V + lex], acc);
      a[tt * D + b] = mk(-f * acc.im, f * acc.re);
    }
  // scaling: the maximum column sum of |A|, from LDS
  if (lane_used)
#pragma unroll
    for (int j = 0; j < NB; ++j) se[mloc][i][j] = mk(sqrt(a[j].re * a[j].re + a[j].im * a[j].im), 0.0);
  __syncthreads();
  double nrm = 0.0;
  for (int j = 0; j < NB; ++j) {
    double sum = 0.0;
    for (int q = 0; q < NB; ++q) sum += se[mloc][q][j].re;
    nrm = sum > nrm ? sum : nrm;
  }
  __syncthreads();
  int sq = 0;
  while (nrm > 0.25 && sq < 60) {
    nrm *= 0.5;
    ++sq;
  }
  int sqmax = sq;   // largest over the wavefront (the block)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const int o = __shfl_xor(sqmax, off, 64);
    sqmax = o > sqmax ? o : sqmax;
  }
  const double sc = ldexp(1.0, -sq);
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    a[j] = sc * a[j];
    om[j] = sc * om[j];
  }
  constexpr int KT = kTaylor;
  cplx<double> e[NB], l[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    e[j] = mk(i == j ? 1.0 : 0.0, 0.0);
    l[j] = mk(0.0, 0.0);
  }
  // e_k = 1 + a e_{k+1} / k,  l_k = (om e_{k+1} + a l_{k+1}) / k
  for (int k = KT; k >= 1; --k) {
    if (lane_used)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        se[mloc][i][j] = e[j];
        sl[mloc][i][j] = l[j];
      }
    __syncthreads();
    const double rk = 1.0 / k;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      cplx<double> ae = mk(0.0, 0.0), al = mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const cplx<double> eq = se[mloc][q][j];
        ae = cfma(a[q], eq, ae);
        al = cfma(om[q], eq, al);
        al = cfma(a[q], sl[mloc][q][j], al);
      }
      e[j] = rk * ae + mk(i == j ? 1.0 : 0.0, 0.0);
      l[j] = rk * al;
    }
    __syncthreads();
  }
  for (int s2 = 0; s2 < sqmax; ++s2) {
    if (lane_used)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        se[mloc][i][j] = e[j];
        sl[mloc][i][j] = l[j];
      }
    __syncthreads();
    cplx<double> te[NB], tl[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      cplx<double> ae = mk(0.0, 0.0), al = mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const cplx<double> eq = se[mloc][q][j];
        ae = cfma(e[q], eq, ae);
        al = cfma(l[q], eq, al);
        al = cfma(e[q], sl[mloc][q][j], al);
      }
      te[j] = ae;
      tl[j] = al;
    }
    if (s2 < sq)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        e[j] = te[j];
        l[j] = tl[j];
      }
    __syncthreads();
  }
  // B' = L(A, B): rows to LDS, then the K entries of the site shared out over
  // the 2 NB lanes of its two matrices (S.v holds 2 sigma)
  if (lane_used)
#pragma unroll
    for (int j = 0; j < NB; ++j) sl[mloc][i][j] = l[j];
  __syncthreads();
  if (valid) {
    const int ml = mloc & ~1;
    for (int idx = c * NB + i; idx < 6 * D * D; idx += 2 * NB) {
      const int p = idx / (D * D), b = (idx / D) % D, a2 = idx % D;
      if (b > a2) continue;
      cplx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int tt = 0; tt < 2; ++tt) acc = cfma(S.v[p][c2][s][tt], sl[ml + c2][tt * D + b][s * D + a2], acc);
      double *k = K + (size_t)p * D * D * V + lex;
      const int e = b == a2 ? b : herm_pair(D, b, a2);
      k[(size_t)e * V] = 0.5 * acc.re;
      if (b != a2) k[(size_t)(e + 1) * V] = 0.5 * acc.im;
    }
  }
}

// Operand of the products below that stays in LDS, 64 lanes side by side.
template <int NB>
struct HermLds {
  cplx<double> *o;   // this lane's upper triangle, 64 entries apart
  double *d;         // and diagonal
  static constexpr int kTri = NB * (NB - 1) / 2;
  __device__ __forceinline__ void put(const Herm<NB> &h, double f) const {
#pragma unroll
    for (int i = 0; i < NB; ++i) d[i * 64] = f * h.d[i];
#pragma unroll
    for (int k = 0; k < kTri; ++k) o[k * 64] = f * h.o[k];
  }
  __device__ __forceinline__ cplx<double> off(int i, int j) const {
    const cplx<double> v = o[Herm<NB>::at(i < j ? i : j, i < j ? j : i) * 64];
    return mk(v.re, i < j ? v.im : -v.im);
  }
};

// r += a b, of whose entries the diagonal's real part and the upper triangle are
// formed: sums of products that are Hermitian as a whole.
template <int NB>
__device__ __forceinline__ void herm_mac(Herm<NB> &r, const HermLds<NB> &a, const Herm<NB> &b) {
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    cplx<double> row[NB];   // row i of a
    const double di = a.d[i * 64];
#pragma unroll
    for (int k = 0; k < NB; ++k) row[k] = k == i ? mk(di, 0.0) : a.off(i, k);
    r.d[i] = fma(di, b.d[i], r.d[i]);
#pragma unroll
    for (int k = 0; k < NB; ++k)
      if (k != i) {
        const cplx<double> y = b.off(i, k);   // b_ki = conj(b_ik)
        r.d[i] = fma(row[k].re, y.re, r.d[i]);
        r.d[i] = fma(row[k].im, y.im, r.d[i]);
      }
#pragma unroll
    for (int j = i + 1; j < NB; ++j) {
      cplx<double> &t = r.o[Herm<NB>::at(i, j)];
      const cplx<double> bij = b.off(i, j);
      t.re = fma(di, bij.re, t.re);
      t.im = fma(di, bij.im, t.im);
      t.re = fma(row[j].re, b.d[j], t.re);
      t.im = fma(row[j].im, b.d[j], t.im);
#pragma unroll
      for (int k = 0; k < NB; ++k)
        if (k != i && k != j) t = cfma(row[k], b.off(k, j), t);
    }
    __builtin_amdgcn_sched_barrier(0);   // one row of a at a time
  }
}

// Exponential form, d_R <= 3: thread per (site, chirality block), the blocks of a
// site in adjacent lanes.  As k_clover_insert with B_c <- L(A_c, B_c) before the K
// entries, L the Frechet derivative of exp at A = C / (4 + m) along B: scaling by
// 2^-s (s from the largest column sum of |A|, down to 1/4), Horner for
// e = exp(A') and its derivative l along B / 2^s (Taylor degree 12, as in the
// field kernels), then s squarings (e, l) <- (e e, l e + e l).  Everything is
// Hermitian (e_k = 1 + A e_{k+1} / k is a real polynomial in A, and
// l_k = (B e_{k+1} + A l_{k+1}) / k its derivative along B), so that a product
// costs its upper triangle; e, l and the sum under way are in registers, A and B
// in LDS.  Bound by FP64 arithmetic at one wavefront per SIMD.  SU(3) FUND 32^4:
// 4.99 ms with a lane per row of a general matrix, 1.94 ms.
template <int D>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1))) void k_clover_insert_exp(
    const cplx<double> *Xe, const cplx<double> *Xo, const cplx<double> *Ye, const cplx<double> *Yo,
    const cplx<double> *__restrict__ clov, const cplx<double> *__restrict__ F, double *__restrict__ K, Geom g,
    SigmaBlocks S, double m0, double csw, double cdet) {
  constexpr int NB = 2 * D, TRI = NB * (NB - 1) / 2;
  __shared__ cplx<double> so[2][TRI * 64];
  __shared__ double sd[2][NB * 64];
  const size_t V = 2 * (size_t)g.Vh;
  const size_t gid = (size_t)blockIdx.x * 64 + threadIdx.x;
  const bool on = gid < 2 * V;   // lanes past the end repeat the last site and store nothing
  const int c = (int)(threadIdx.x & 1);
  const unsigned lex = (unsigned)((on ? gid : 2 * V - 2) >> 1);
  unsigned r = lex;
  const int z = (int)(r % g.Z); r /= g.Z;
  const int y = (int)(r % g.Y); r /= g.Y;
  const int x = (int)(r % g.X);
  const int t = (int)(r / g.X);
  const int par = (t + x + y + z) & 1;
  const size_t cb = lex >> 1;
  const HermLds<NB> A{so[0] + threadIdx.x, sd[0] + threadIdx.x}, B{so[1] + threadIdx.x, sd[1] + threadIdx.x};
  int sq;
  {
    // A = (i/4) c_sw sum_p S[p][c] F_p / (4 + m)
    const double f = 0.25 * csw / (4.0 + m0);
    Herm<NB> a;
#pragma unroll
    for (int i = 0; i < NB; ++i) a.d[i] = 0.0;
#pragma unroll
    for (int k = 0; k < TRI; ++k) a.o[k] = mk(0.0, 0.0);
#pragma unroll
    for (int p = 0; p < 6; ++p) {
      cplx<double> fp[D][D];
#pragma unroll
      for (int i = 0; i < D; ++i)
#pragma unroll
        for (int j = 0; j < D; ++j) fp[i][j] = F[((size_t)p * D * D + i * D + j) * V + lex];
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int tt = s2; tt < 2; ++tt) {
          const cplx<double> sv = S.v[p][c][s2][tt];
#pragma unroll
          for (int i2 = 0; i2 < D; ++i2)
#pragma unroll
            for (int j2 = 0; j2 < D; ++j2) {
              const int i = s2 * D + i2, j = tt * D + j2;
              if (i == j) {   // Re(i sv fp) = -Im(sv fp)
                a.d[i] = fma(-sv.re, fp[i2][j2].im, a.d[i]);
                a.d[i] = fma(-sv.im, fp[i2][j2].re, a.d[i]);
              } else if (i < j) {
                cplx<double> &o = a.o[Herm<NB>::at(i, j)];
                o = cfma(mk(-sv.im, sv.re), fp[i2][j2], o);
              }
            }
        }
      __builtin_amdgcn_sched_barrier(0);   // one plane's F entries at a time
    }
    double nrm = 0.0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      double sum = fabs(a.d[i]);
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (j != i) {
          const cplx<double> v = a.off(i, j);
          sum += sqrt(v.re * v.re + v.im * v.im);
        }
      nrm = sum > nrm ? sum : nrm;
    }
    sq = exp_squarings(nrm * fabs(f));
    A.put(a, ldexp(f, -sq));
  }
  {
    Herm<NB> b;
    const cplx<double> *X = par ? Xo : Xe, *Y = par ? Yo : Ye;
    const cplx<double> *Mi = clov + (size_t)(2 + c) * (NB * (NB + 1) / 2) * g.stride + cb;
    cplx<double> xv[NB], yv[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const size_t o = (size_t)(2 * c * D + k) * g.stride + cb;
      xv[k] = Xe ? X[o] : mk(0.0, 0.0);
      yv[k] = Xe ? Y[o] : mk(0.0, 0.0);
    }
    const double w = par == 1 ? 2.0 * cdet : 0.0;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = i; j < NB; ++j) {   // x_i conj(y_j) + y_i conj(x_j), + 2 cdet D_oo^{-1}
        cplx<double> v = cfma_conj(xv[j], yv[i], cfma_conj(yv[j], xv[i], mk(0.0, 0.0)));
        if (w != 0.0) v = v + w * Mi[(size_t)tri_index(NB, i, j) * g.stride];
        if (i == j) b.d[i] = v.re;
        else b.o[Herm<NB>::at(i, j)] = v;
      }
    B.put(b, ldexp(1.0, -sq));
  }
  // e_k = 1 + A e_{k+1} / k,  l_k = (B e_{k+1} + A l_{k+1}) / k, from e = 1, l = 0
  Herm<NB> e, l;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    e.d[i] = 1.0;
    l.d[i] = 0.0;
  }
#pragma unroll
  for (int k = 0; k < TRI; ++k) e.o[k] = l.o[k] = mk(0.0, 0.0);
#pragma unroll 1
  for (int k = kTaylor; k >= 1; --k) {
    const double rk = 1.0 / k;
    Herm<NB> n;
#pragma unroll
    for (int i = 0; i < NB; ++i) n.d[i] = 0.0;
#pragma unroll
    for (int q = 0; q < TRI; ++q) n.o[q] = mk(0.0, 0.0);
    herm_mac<NB>(n, A, l);
    herm_mac<NB>(n, B, e);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      l.d[i] = rk * n.d[i];
      n.d[i] = 0.0;
    }
#pragma unroll
    for (int q = 0; q < TRI; ++q) {
      l.o[q] = rk * n.o[q];
      n.o[q] = mk(0.0, 0.0);
    }
    herm_mac<NB>(n, A, e);
#pragma unroll
    for (int i = 0; i < NB; ++i) e.d[i] = fma(rk, n.d[i], 1.0);
#pragma unroll
    for (int q = 0; q < TRI; ++q) e.o[q] = rk * n.o[q];
  }
#pragma unroll 1
  for (int q = 0; q < sq; ++q) {
    Herm<NB> n;   // e l + l e: (e l)_ij + conj((e l)_ji)
#pragma unroll
    for (int i = 0; i < NB; ++i) n.d[i] = 0.0;
#pragma unroll
    for (int k = 0; k < TRI; ++k) n.o[k] = mk(0.0, 0.0);
    A.put(e, 1.0);   // (A and B are done with)
    B.put(l, 1.0);
    herm_mac<NB>(n, A, l);
    herm_mac<NB>(n, B, e);
    l = n;
#pragma unroll
    for (int i = 0; i < NB; ++i) n.d[i] = 0.0;
#pragma unroll
    for (int k = 0; k < TRI; ++k) n.o[k] = mk(0.0, 0.0);
    herm_mac<NB>(n, A, e);
    e = n;
  }
  // K entries of the site, the two blocks' halves added across the lane pair
  // (S.v holds 2 sigma)
#pragma unroll 1
  for (int p = 0; p < 6; ++p) {
    const cplx<double> s00 = S.v[p][c][0][0], s01 = S.v[p][c][0][1], s10 = S.v[p][c][1][0], s11 = S.v[p][c][1][1];
    double *k = K + (size_t)p * D * D * V + lex;
#pragma unroll
    for (int b = 0; b < D; ++b)
#pragma unroll
      for (int a2 = b; a2 < D; ++a2) {
        // sum_st sigma_st (B_c)_(t b),(s a)
        const auto ent = [&](int i, int j) { return i == j ? mk(l.d[i], 0.0) : l.off(i, j); };
        cplx<double> v = cfma(s00, ent(b, a2), mk(0.0, 0.0));
        v = cfma(s01, ent(D + b, a2), v);
        v = cfma(s10, ent(b, D + a2), v);
        v = cfma(s11, ent(D + b, D + a2), v);
        v.re += __shfl_xor(v.re, 1, 64);
        v.im += __shfl_xor(v.im, 1, 64);
        const int q = b == a2 ? b : herm_pair(D, b, a2);
        if (on && c == 0) k[(size_t)q * V] = 0.5 * v.re;
        if (on && c == 1 && b != a2) k[(size_t)(q + 1) * V] = 0.5 * v.im;
      }
  }
}

// The Hermitian matrix `m` of a scratch array (K: m = plane; G: m = 4 plane +
// leaf) at site xl from its n^2 stored reals.
template <int N>
__device__ __forceinline__ void herm_load(cplx<double> (&gm)[N][N], const double *G, int m, unsigned xl, size_t V) {
  const double *gr = G + (size_t)__builtin_amdgcn_readfirstlane(m) * N * N * V;
#pragma unroll
  for (int i = 0; i < N; ++i) gm[i][i] = mk(*at(gr + (size_t)i * V, xl), 0.0);
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = i + 1; j < N; ++j) {
      const int e = herm_pair(N, i, j);
      const double re = *at(gr + (size_t)e * V, xl), im = *at(gr + (size_t)(e + 1) * V, xl);
      gm[i][j] = mk(re, im);
      gm[j][i] = mk(re, -im);
    }
}

// Thread per (plane p, site x): for the four leaves l of Q_p(x), the matrix
// g = sum_b Re tr[T^b_R R(l) K_p] T^b = (H - tr(H)/N)/2 with H the Hermitian
// part of the pull-back of R(l) K_p, into G[p][k][N][N][V].
template <int N, int REP>
__global__ __launch_bounds__(64) void k_clover_leafgen(const cplx<double> *__restrict__ U,
                                                       const double *__restrict__ K,
                                                       double *__restrict__ G, Geom g) {
  constexpr int D = rep_dim(N, REP);
  const size_t V = 2 * (size_t)g.Vh;
  const unsigned gid = xcd_block(blockIdx.x, gridDim.x) * 64u + threadIdx.x;
  // 64-site chunks, the six planes of a chunk in consecutive wavefronts (the
  // planes that share a link direction read it close together in time)
  const unsigned chunk = gid / 384u;
  const int r6 = (int)(gid - chunk * 384u);
  const int p = __builtin_amdgcn_readfirstlane(r6 >> 6);
  const unsigned lex = chunk * 64u + (r6 & 63);
  if (lex >= V) return;
  int mu, nu;
  plane_dirs(p, mu, nu);
  int c[4];
  lex_coords(g, lex, c);
  const PlaneNb pn(g, c, lex, mu, nu);
  cplx<double> Kh[D][D];
  herm_load<D>(Kh, K, p, lex, V);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    cplx<double> L[N][N];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const LeafStep s = kLeafC[k][f];
      cplx<double> u[N][N];
      load_link<N>(u, U, V, pn.at(s.a, s.b), s.dir ? nu : mu, s.dag != 0);
      if (f == 0) {
        for (int i = 0; i < N; ++i)
          for (int j = 0; j < N; ++j) L[i][j] = u[i][j];
      } else {
        mul_right<N>(L, u);
      }
    }
    cplx<double> R[D][D], M[D][D];
    for (int A = 0; A < D; ++A)
      for (int B = 0; B < D; ++B) R[A][B] = rep_entry<N, REP>(L, A, B);
    for (int A = 0; A < D; ++A)
      for (int B = 0; B < D; ++B) {
        cplx<double> sum = mk(0.0, 0.0);
        for (int C = 0; C < D; ++C) sum = cfma(R[A][C], Kh[C][B], sum);
        M[A][B] = sum;
      }
    cplx<double> Z[N][N];
    rep_pullback<N, REP>([&](int B, int A) { return M[B][A]; }, Z);
    double tr = 0.0;
    for (int i = 0; i < N; ++i) tr += Z[i][i].re;
    // g = (H - tr(H)/N) / 2, H = (Z + Z^+)/2, Hermitian: stored as N^2 reals
    // (g_ii, then Re g_ij and Im g_ij for i < j), see herm_load
    double *gr = G + (size_t)(p * 4 + k) * N * N * V;
#pragma unroll
    for (int i = 0; i < N; ++i) *at(gr + (size_t)i * V, lex) = 0.5 * (Z[i][i].re - tr / N);
    int t = N;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = i + 1; j < N; ++j) {
        *at(gr + (size_t)t * V, lex) = 0.25 * (Z[i][j].re + Z[j][i].re);
        *at(gr + (size_t)(t + 1) * V, lex) = 0.25 * (Z[i][j].im - Z[j][i].im);
        t += 2;
      }
  }
}

// X <- S^+ X S for a Hermitian X, S a fundamental link (dag: its adjoint)
// read from the structure-of-arrays copy; the upper triangle is formed and
// mirrored, so X stays exactly Hermitian.
template <int N>
__device__ __forceinline__ void herm_transport(cplx<double> (&X)[N][N], const cplx<double> *Us, size_t V, unsigned lex,
                                               int mu, bool dag) {
  cplx<double> S[N][N], T[N][N];
  load_link<N>(S, Us, V, lex, mu, dag);
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      cplx<double> s = mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < N; ++q) s = cfma(X[i][q], S[q][j], s);
      T[i][j] = s;
    }
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = i; j < N; ++j) {
      cplx<double> s = mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < N; ++q) s = cfma_conj(S[q][i], T[q][j], s);
      X[i][j] = i == j ? mk(s.re, 0.0) : s;
      if (j != i) X[j][i] = mk(s.re, -s.im);
    }
}

// The plaquette of plane p = (lo, hi) with lower corner z (offsets za, zb
// along lo, hi from y), traversed lo, hi, lo^+, hi^+: steps S_0 = U_lo(z),
// S_1 = U_hi(z+lo), S_2 = U_lo(z+hi)^+, S_3 = U_hi(z)^+, corners c_m = start
// of S_m.  The leaf k of a site is this loop started at c_k (leaf 0 at z,
// 1 at z+lo, 2 at z+lo+hi, 3 at z+hi), so for the link at step J every leaf
// of the plaquette contributes B^+ g_k B with B the path from c_k to step J,
// and the four nest as
//   H_J = g_J + S_{J+3}^+ [g_{J+3} + S_{J+2}^+ [g_{J+2} + S_{J+1}^+ g_{J+1} S_{J+1}] S_{J+2}] S_{J+3}
// (indices mod 4): three transports instead of four separate paths.  The
// link at a forward step receives +H_J, at a backward one -S_J^+ H_J S_J.
template <int N, int J>
__device__ __forceinline__ void plaquette_horner(cplx<double> (&acc)[N][N], const cplx<double> *Us,
                                                 const double *Gl, size_t V, const PlaneNb &pn, int lo, int hi,
                                                 int p, int za, int zb) {
  constexpr int ca[4] = {0, 1, 1, 0}, cb[4] = {0, 0, 1, 1};   // corner c_m - z
  constexpr int sa[4] = {0, 1, 0, 0}, sb[4] = {0, 0, 1, 0};   // start of the link of S_m - z
  cplx<double> H[N][N], gm[N][N];
#pragma unroll
  for (int s = 1; s <= 3; ++s) {
    const int m = (J + s) & 3;
    herm_load<N>(gm, Gl, p * 4 + m, pn.at(za + ca[m], zb + cb[m]), V);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) H[i][j] = s == 1 ? gm[i][j] : H[i][j] + gm[i][j];
    herm_transport<N>(H, Us, V, pn.at(za + sa[m], zb + sb[m]), (m & 1) ? hi : lo, m >= 2);
  }
  herm_load<N>(gm, Gl, p * 4 + J, pn.at(za + ca[J], zb + cb[J]), V);
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) acc[i][j] = acc[i][j] + H[i][j] + gm[i][j];
}

// Thread per link (y, rho): P = coef sum over the planes (rho, nu) of the
// contributions of the two plaquettes that hold the link (see
// plaquette_horner); out as in the hopping force: P, or G = 2i P U
// (gradient), stored or accumulated.
template <int N>
__global__ __launch_bounds__(128) void k_clover_gather(const cplx<double> *__restrict__ U,
                                                       const double *__restrict__ Gl, double *P, Geom g,
                                                       double coef, int gradient, int accumulate) {
  const size_t V = 2 * (size_t)g.Vh;
  const unsigned gid = xcd_block(blockIdx.x, gridDim.x) * 128u + threadIdx.x;
  // 64-site chunks, the four directions of a chunk in consecutive
  // wavefronts: the lanes of a wavefront hold one direction on consecutive
  // sites (coalesced structure-of-arrays link reads, the same planes in every
  // lane), and the two directions of a plane read its leaf matrices close
  // together in time
  const unsigned chunk = gid / 256u;
  const int r4 = (int)(gid & 255u);
  const int rho = __builtin_amdgcn_readfirstlane(r4 >> 6);
  const unsigned lex = chunk * 64u + (r4 & 63);
  if (lex >= V) return;
  int cy[4];
  lex_coords(g, lex, cy);
  // forward (af) and backward (ab) occurrences; the backward sum is
  // transported by the link itself once at the end
  cplx<double> af[N][N], ab[N][N];
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) af[i][j] = ab[i][j] = mk(0.0, 0.0);
  for (int nu = 0; nu < 4; ++nu) {
    if (nu == rho) continue;
    const int lo = rho < nu ? rho : nu, hi = rho < nu ? nu : rho;
    const int p = lo == 0 ? hi - 1 : lo == 1 ? hi + 1 : 5;
    const PlaneNb pn(g, cy, lex, lo, hi);
    if (rho == lo) {
      plaquette_horner<N, 0>(af, U, Gl, V, pn, lo, hi, p, 0, 0);    // S_0 of the plaquette at y
      plaquette_horner<N, 2>(ab, U, Gl, V, pn, lo, hi, p, 0, -1);   // S_2 of the one at y - hi
    } else {
      plaquette_horner<N, 1>(af, U, Gl, V, pn, lo, hi, p, -1, 0);   // S_1 of the one at y - lo
      plaquette_horner<N, 3>(ab, U, Gl, V, pn, lo, hi, p, 0, 0);    // S_3 of the one at y
    }
  }
  // S_J = U_rho(y)^+ for the backward steps: S_J^+ ab S_J = U ab U^+
  herm_transport<N>(ab, U, V, lex, rho, true);
  cplx<double> acc[N][N];
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) acc[i][j] = af[i][j] - ab[i][j];
  cplx<double> Fo[N][N];
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) Fo[i][j] = coef * acc[i][j];
  if (gradient) {
    const cplx<double> *u = U + (size_t)rho * N * N * V + lex;
    cplx<double> Gm[N][N];
    for (int i = 0; i < N; ++i)
      for (int j = 0; j < N; ++j) {
        cplx<double> s = mk(0.0, 0.0);
        for (int q = 0; q < N; ++q) s = cfma(Fo[i][q], u[(size_t)(q * N + j) * V], s);
        Gm[i][j] = mk(-2.0 * s.im, 2.0 * s.re);
      }
    for (int i = 0; i < N; ++i)
      for (int j = 0; j < N; ++j) Fo[i][j] = Gm[i][j];
  }
  double *out = P + ((size_t)lex * 4 + rho) * N * N * 2;
  for (int i = 0; i < N; ++i)
    for (int j = 0; j < N; ++j) {
      double re = Fo[i][j].re, im = Fo[i][j].im;
      if (accumulate) {
        re += out[2 * (i * N + j)];
        im += out[2 * (i * N + j) + 1];
      }
      out[2 * (i * N + j)] = re;
      out[2 * (i * N + j) + 1] = im;
    }
}

// Fundamental representation: the link force without leaf matrices.  A leaf
// whose loop starts at corner c_k passes the link as B U rest, and moving the
// link moves Im tr[B U rest K_k] by Re tr[T U rest K_k B]: the link at step J
// of the plaquette S_0 S_1 S_2 S_3 (see plaquette_horner) receives
//   U R_J,   R_J = sum_k S_{J+1}..S_{k-1} K_k S_k..S_{J+3}   (k = J+1 .. J+4),
// the sum over the corners of the plaquette, and a backward step, as U^+ in
// the loop, -R_J U^+.  With a = S_{J+1}, A = a, M = K a each further corner is
// M <- (M + A K) S, A <- A S: eight products for the four corners, and the
// Hermitian traceless part is taken once, of the sum over the plaquettes.
template <int N>
__device__ __forceinline__ void herm_mac(cplx<double> (&M)[N][N], const cplx<double> (&A)[N][N],
                                         const cplx<double> (&K)[N][N]) {   // M += A K, K Hermitian
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      cplx<double> s = rfma(K[j][j].re, A[i][j], M[i][j]);
#pragma unroll
      for (int q = 0; q < N; ++q)
        if (q != j) s = cfma(A[i][q], K[q][j], s);
      M[i][j] = s;
    }
}

// off, not known before d is: loads from it are not issued earlier.  (The
// compiler otherwise issues the loads of all steps at once, and spills.)
__device__ __forceinline__ unsigned after(unsigned off, double d) {
  asm volatile("" : "+v"(off) : "v"(d));
  return off;
}

// R_J of one plaquette; the loads of a step are issued one step ahead.
template <int N, int J>
__device__ __forceinline__ void plaquette_corners(cplx<double> (&M)[N][N], const cplx<double> *Us, const double *K,
                                                  size_t V, const PlaneNb &pn, int lo, int hi, int p, int za, int zb) {
  constexpr int ca[4] = {0, 1, 1, 0}, cb[4] = {0, 0, 1, 1};   // corner c_m - z
  constexpr int sa[4] = {0, 1, 0, 0}, sb[4] = {0, 0, 1, 0};   // start of the link of S_m - z
  constexpr int m1 = (J + 1) & 3, m2 = (J + 2) & 3, m3 = (J + 3) & 3;
  cplx<double> A[N][N], S2[N][N], k2[N][N], S3[N][N], k3[N][N], kJ[N][N];
  load_link<N>(A, Us, V, pn.at(za + sa[m1], zb + sb[m1]), (m1 & 1) ? hi : lo, m1 >= 2);
  herm_load<N>(M, K, p, pn.at(za + ca[m1], zb + cb[m1]), V);
  load_link<N>(S2, Us, V, pn.at(za + sa[m2], zb + sb[m2]), (m2 & 1) ? hi : lo, m2 >= 2);
  herm_load<N>(k2, K, p, pn.at(za + ca[m2], zb + cb[m2]), V);
  mul_right<N>(M, A);
  load_link<N>(S3, Us, V, after(pn.at(za + sa[m3], zb + sb[m3]), M[0][0].re), (m3 & 1) ? hi : lo, m3 >= 2);
  herm_load<N>(k3, K, p, after(pn.at(za + ca[m3], zb + cb[m3]), M[0][0].re), V);
  herm_mac<N>(M, A, k2);
  mul_right<N>(M, S2);
  mul_right<N>(A, S2);
  herm_load<N>(kJ, K, p, after(pn.at(za + ca[J], zb + cb[J]), M[0][0].re), V);
  herm_mac<N>(M, A, k3);
  mul_right<N>(M, S3);
  mul_right<N>(A, S3);
  herm_mac<N>(M, A, kJ);
}

// Thread per link (y, rho) as k_clover_gather, with which it shares the order
// of work; a block holds the four directions of 64 sites.  Bound by its loads
// of neighbour links and K through L2 (19 links and 24 K a link) at two waves
// per SIMD.  SU(3) FUND 24^4: 612 us with the leaf matrices, after 484 us to
// make them (573 MB of scratch against K's 143 MB); 579 us from K.
template <int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(N <= 3 ? 2 : 1))) void k_clover_gather_fund(const cplx<double> *__restrict__ U,
                                                            const double *__restrict__ K, double *P, Geom g,
                                                            double coef, int gradient, int accumulate) {
  __shared__ cplx<double> acc[2 * N * N][256];
  const size_t V = 2 * (size_t)g.Vh;
  const unsigned b = xcd_block(blockIdx.x, gridDim.x);
  const int rho = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const unsigned lex = b * 64u + (threadIdx.x & 63);
  if (lex >= V) return;
  int cy[4];
  lex_coords(g, lex, cy);
  // af, ab: the sums over the plaquettes that pass the link forward and
  // backward, each thread's own in LDS (they leave room for the products)
#pragma unroll
  for (int e = 0; e < 2 * N * N; ++e) acc[e][threadIdx.x] = mk(0.0, 0.0);
#pragma unroll 1
  for (int q = 0; q < 8; ++q) {
    const int nu = q & 3, back = q >> 2;
    if (nu == rho) continue;
    const int lo = rho < nu ? rho : nu, hi = rho < nu ? nu : rho;
    const int p = lo == 0 ? hi - 1 : lo == 1 ? hi + 1 : 5;
    const PlaneNb pn(g, cy, lex, lo, hi);
    cplx<double> M[N][N];
    if (rho == lo) {
      if (!back) plaquette_corners<N, 0>(M, U, K, V, pn, lo, hi, p, 0, 0);   // S_0 of the plaquette at y
      else plaquette_corners<N, 2>(M, U, K, V, pn, lo, hi, p, 0, -1);        // S_2 of the one at y - hi
    } else {
      if (!back) plaquette_corners<N, 1>(M, U, K, V, pn, lo, hi, p, -1, 0);  // S_1 of the one at y - lo
      else plaquette_corners<N, 3>(M, U, K, V, pn, lo, hi, p, 0, 0);         // S_3 of the one at y
    }
    cplx<double>(*s)[256] = acc + back * N * N;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) s[i * N + j][threadIdx.x] = s[i * N + j][threadIdx.x] + M[i][j];
  }
  // H: Hermitian part of Z = U af - ab U^+ (upper triangle)
  cplx<double> H[N][N], u[N][N];
  load_link<N>(u, U, V, lex, rho, false);
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = i; j < N; ++j) {
      cplx<double> s = mk(0.0, 0.0), t = s;   // Z_ij and Z_ji
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const cplx<double> bi = acc[N * N + i * N + q][threadIdx.x];
        s = cfma(u[i][q], acc[q * N + j][threadIdx.x], s);
        s = cfma_conj(u[j][q], mk(-bi.re, -bi.im), s);
        if (j != i) {
          const cplx<double> bj = acc[N * N + j * N + q][threadIdx.x];
          t = cfma(u[j][q], acc[q * N + i][threadIdx.x], t);
          t = cfma_conj(u[i][q], mk(-bj.re, -bj.im), t);
        }
      }
      if (j == i) t = s;
      H[i][j] = mk(0.5 * (s.re + t.re), 0.5 * (s.im - t.im));
    }
  // force = coef (H - tr(H)/N) / 2
  double tr = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) tr += H[i][i].re;
  cplx<double> Fo[N][N];
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = i; j < N; ++j) {
      Fo[i][j] = mk(0.5 * coef * (H[i][j].re - (i == j ? tr / N : 0.0)), 0.5 * coef * H[i][j].im);
      if (j != i) Fo[j][i] = mk(Fo[i][j].re, -Fo[i][j].im);
    }
  if (gradient) {
    cplx<double> Gm[N][N];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) {
        cplx<double> s = mk(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < N; ++q) s = cfma(Fo[i][q], u[q][j], s);
        Gm[i][j] = mk(-2.0 * s.im, 2.0 * s.re);
      }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) Fo[i][j] = Gm[i][j];
  }
  cplx<double> *out = reinterpret_cast<cplx<double> *>(P) + ((size_t)lex * 4 + rho) * N * N;
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) {
      cplx<double> v = Fo[i][j];
      if (accumulate) v = v + out[i * N + j];
      out[i * N + j] = v;
    }
}

// log|det D_oo(x)| summed over the odd sites: thread per (odd site, block),
// the block index fastest, Gaussian elimination with partial pivoting of the
// stored inverse block (log|det D_oo| = -log|det D_oo^{-1}|) in registers (row
// interchanges as selects, every index a compile-time constant), block partial
// sums.  SU(3) FUND 24^4: 206 us with indexed rows, which went to scratch;
// the whole call 233 us then, 57 us now.
template <int D>
__global__ __launch_bounds__(64) void k_clover_logdet(const cplx<double> *__restrict__ clov, double *partial,
                                                      Geom g) {
  constexpr int NB = 2 * D;
  const unsigned gid = blockIdx.x * 64u + threadIdx.x;
  double v = 0.0;
  if (gid < 2 * (unsigned)g.Vh) {
    const unsigned c = gid & 1, cb = gid >> 1;
    const cplx<double> *Mi = clov + (size_t)(2 + c) * (NB * (NB + 1) / 2) * g.stride + cb;
    cplx<double> a[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = i; j < NB; ++j) {
        const cplx<double> m = Mi[(size_t)tri_index(NB, i, j) * g.stride];
        a[i][j] = m;
        if (j != i) a[j][i] = mk(m.re, -m.im);
      }
    double ld = 0.0;
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      int p = k;
      double best = a[k][k].re * a[k][k].re + a[k][k].im * a[k][k].im;
#pragma unroll
      for (int r = k + 1; r < NB; ++r) {
        const double m2 = a[r][k].re * a[r][k].re + a[r][k].im * a[r][k].im;
        p = m2 > best ? r : p;
        best = m2 > best ? m2 : best;
      }
      ld += 0.5 * log(best);
#pragma unroll
      for (int r = k + 1; r < NB; ++r) {
        const bool sw = p == r;
#pragma unroll
        for (int j = k; j < NB; ++j) {
          const cplx<double> tk = a[k][j], tr = a[r][j];
          a[k][j] = sw ? tr : tk;
          a[r][j] = sw ? tk : tr;
        }
      }
      const double dn = 1.0 / best;
      const cplx<double> di = mk(a[k][k].re * dn, -a[k][k].im * dn);
#pragma unroll
      for (int r = k + 1; r < NB; ++r) {
        const cplx<double> f = cmul(a[r][k], di);
#pragma unroll
        for (int j = k + 1; j < NB; ++j) a[r][j] = a[r][j] - cmul(f, a[k][j]);
      }
    }
    v = -ld;
  }
  const double s = wave_sum(v);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The same for larger blocks, NB lanes per matrix (rows_exchange), the 64
// matrices of a block in turn.
template <int D>
__global__ __launch_bounds__(64) void k_clover_logdet_rows(const cplx<double> *__restrict__ clov, double *partial,
                                                           Geom g) {
  constexpr int NB = 2 * D, MPB = 64 / NB;
  __shared__ cplx<double> sh[MPB][NB][NB + 1];
  __shared__ int perm[MPB][NB];
  const int mloc0 = (int)threadIdx.x / NB;
  const bool lane_used = mloc0 < MPB;
  const int mloc = lane_used ? mloc0 : MPB - 1;
  const int i = lane_used ? (int)threadIdx.x - mloc * NB : 0;
  const unsigned n = 2 * (unsigned)g.Vh;
  double v = 0.0;
  for (int m0 = 0; m0 < 64; m0 += MPB) {
    const unsigned gid = blockIdx.x * 64u + m0 + mloc;
    const bool valid = lane_used && m0 + mloc < 64 && gid < n;
    const unsigned m = valid ? gid : 0;
    const unsigned c = m & 1, cb = m >> 1;
    const cplx<double> *Mi = clov + (size_t)(2 + c) * (NB * (NB + 1) / 2) * g.stride + cb;
    cplx<double> w[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) w[j] = herm_entry(Mi, g.stride, NB, i, j);
    int mine;
    const double ld = rows_exchange<NB>(w, sh[mloc], perm[mloc], i, lane_used, mine);
    if (valid && i == 0) v -= ld;
  }
  const double s = wave_sum(v);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

constexpr bool clover_rep_ok(int N, int REP) {
  return (REP != 3 || N > 2) && (rep_dim(N, REP) == 2 || rep_dim(N, REP) == 3 || rep_dim(N, REP) == 4 ||
                                 rep_dim(N, REP) == 6);
}

template <int N, int REP>
static hipError_t clover_force_nr(void *P, const void *Xe, const void *Xo, const void *Ye, const void *Yo,
                                  const void *U0, const void *clov, double *F, double *K, double *Gl, double *Us,
                                  const Geom &g,
                                  double m0, double csw, int expo, double cdet, double coef, int gradient,
                                  int accumulate, hipStream_t st) {
  if constexpr (clover_rep_ok(N, REP)) {
    constexpr int D = rep_dim(N, REP);
    const size_t V = 2 * (size_t)g.Vh;
    {
      hipError_t e = links_soa_launch<N>(U0, Us, g, st);
      if (e != hipSuccess) return e;
    }
    const double *U = Us;
    if (expo) {
      hipError_t e = F_launch<N, REP>(U, F, g, st);
      if (e != hipSuccess) return e;
    }
    const SigmaBlocks S = sigma_blocks();
    const dim3 ig((unsigned)((V + 63) / 64));
    const cplx<double> *xe = (const cplx<double> *)Xe, *xo = (const cplx<double> *)Xo, *ye = (const cplx<double> *)Ye,
                       *yo = (const cplx<double> *)Yo, *cl = (const cplx<double> *)clov, *u = (const cplx<double> *)U;
    if (expo) {
      if constexpr (D <= 3) {
        hipLaunchKernelGGL((k_clover_insert_exp<D>), dim3((unsigned)((2 * V + 63) / 64)), dim3(64), 0, st, xe, xo, ye,
                           yo, cl, (const cplx<double> *)F, K, g, S, m0, csw, cdet);
      } else {
        constexpr int MPB = 64 / (2 * D) / 2 * 2;
        const dim3 rg((unsigned)((2 * V + MPB - 1) / MPB));
        hipLaunchKernelGGL((k_clover_insert_rows<D>), rg, dim3(64), 0, st, xe, xo, ye, yo, cl,
                           (const cplx<double> *)F, K, g, S, m0, csw, cdet);
      }
    } else if (Xe) {
      hipLaunchKernelGGL((k_clover_insert<D, false>), ig, dim3(64), 0, st, xe, xo, ye, yo, cl, K, g, S, cdet);
    } else {
      hipLaunchKernelGGL((k_clover_insert<D, true>), ig, dim3(64), 0, st, xe, xo, ye, yo, cl, K, g, S, cdet);
    }
    if constexpr (REP == 0) {
      hipLaunchKernelGGL((k_clover_gather_fund<N>), ig, dim3(256), 0, st, u, K, (double *)P, g, coef, gradient,
                         accumulate);
    } else {
      hipLaunchKernelGGL((k_clover_leafgen<N, REP>), dim3((unsigned)(6 * ((V + 63) / 64))), dim3(64), 0, st, u, K, Gl,
                         g);
      hipLaunchKernelGGL((k_clover_gather<N>), dim3((unsigned)(2 * ((V + 63) / 64))), dim3(128), 0, st, u, Gl,
                         (double *)P, g, coef, gradient, accumulate);
    }
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <int N>
static hipError_t clover_force_n(void *P, const void *Xe, const void *Xo, const void *Ye, const void *Yo,
                                 const void *U, const void *clov, double *F, double *K, double *Gl, double *Us,
                                 const Geom &g,
                                 int rep, double m0, double csw, int expo, double cdet, double coef, int gradient,
                                 int accumulate, hipStream_t st) {
  switch (rep) {
    case 0: return clover_force_nr<N, 0>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, m0, csw, expo, cdet, coef, gradient, accumulate, st);
    case 1: return clover_force_nr<N, 1>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, m0, csw, expo, cdet, coef, gradient, accumulate, st);
    case 2: return clover_force_nr<N, 2>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, m0, csw, expo, cdet, coef, gradient, accumulate, st);
    case 3: return clover_force_nr<N, 3>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, m0, csw, expo, cdet, coef, gradient, accumulate, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_clover_force(void *P, const void *Xe, const void *Xo, const void *Ye, const void *Yo, const void *U,
                               const void *clov, double *F, double *K, double *Gl, double *Us, const Geom &g, int N, int rep,
                               double m0, double csw, int expo, double cdet, double coef, int gradient, int accumulate,
                               hipStream_t st) {
  switch (N) {
    case 2: return clover_force_n<2>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, rep, m0, csw, expo, cdet, coef, gradient, accumulate, st);
    case 3: return clover_force_n<3>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, rep, m0, csw, expo, cdet, coef, gradient, accumulate, st);
    case 4: return clover_force_n<4>(P, Xe, Xo, Ye, Yo, U, clov, F, K, Gl, Us, g, rep, m0, csw, expo, cdet, coef, gradient, accumulate, st);
  }
  return hipErrorInvalidValue;
}

int clover_logdet_blocks(const Geom &g) { return (int)((2 * (size_t)g.Vh + 63) / 64); }

hipError_t launch_clover_logdet(const void *clov, double *partial, const Geom &g, int d, hipStream_t st) {
  const dim3 grid((unsigned)clover_logdet_blocks(g));
  switch (d) {
    case 2: hipLaunchKernelGGL(k_clover_logdet<2>, grid, dim3(64), 0, st, (const cplx<double> *)clov, partial, g); break;
    case 3: hipLaunchKernelGGL(k_clover_logdet<3>, grid, dim3(64), 0, st, (const cplx<double> *)clov, partial, g); break;
    case 4: hipLaunchKernelGGL(k_clover_logdet_rows<4>, grid, dim3(64), 0, st, (const cplx<double> *)clov, partial, g); break;
    case 6: hipLaunchKernelGGL(k_clover_logdet_rows<6>, grid, dim3(64), 0, st, (const cplx<double> *)clov, partial, g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace wd
