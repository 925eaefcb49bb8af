// Host-side launchers of the libwdirac kernels (internal interface).
//
// A context holds one lattice or a batch of up to MAXLAT lattices of
// different shapes (each with its own geometry).  Packed fields of a batch are
// the concatenation of the per-lattice fields, lattice by lattice.  A
// "system" is one independent field of a packed object: a right-hand side of
// a single lattice, or one lattice of a batch (batches carry one right-hand
// side).  Reductions and CG scalars are per system.
#pragma once

#include <hip/hip_runtime.h>

#include "wd_common.h"

namespace wd {

constexpr int MAXSYS = 12;
constexpr int MAXLAT = 8;

// HOP_COMPACT / HOP_COMPACT_PAIR: the colour-split forms reading the
// fundamental links and rebuilding the two-index represented entries in
// registers (SYM and 2AS only, where N^2 < d_R^2).
// HOP_COLOUR_QUAD: the colour-split form staging two directions (four hops)
// per barrier phase (one rhs per block, d_R <= 4).
// HOP_MULTI: several right-hand sides per block, one wavefront each, with the
// tile's link entries staged once per block in LDS (hop_mr.hip).
enum {
  HOP_SITE = 0,
  HOP_COLOUR = 1,
  HOP_COLOUR_PAIR = 2,
  HOP_COMPACT = 3,
  HOP_COMPACT_PAIR = 4,
  HOP_COLOUR_QUAD = 5,
  HOP_MULTI = 6
};

// One lattice of a launch.
struct LatDesc {
  Geom g;
  int tile0;        // first tile of this lattice in the launch (set by the launcher)
  int ntiles;       // tiles of this lattice (set by the launcher)
  long long soff;   // offset of this lattice in packed half spinors, complex elements
  long long loff;   // offset of this lattice in packed links, link elements
  long long floff;  // offset of this lattice in the compact fundamental links, complex elements
};

// Number of valid partial sums per system (rows of a [system][prow] array).
struct Counts {
  int n[MAXSYS];
};

// CG (see api.hip for the algorithm).  One record per system.  rho, active,
// iters, status, need_update and rmax are the state the host reads: written
// by k_cg_restart and at the end of an iteration (cg_end_step).  rho_it and act_it
// are their copies for the iteration under way (cg_alpha_step), read by every
// block of the kernels that follow while the state is being rewritten.
struct CgScalars {
  double rho;       // <r, r>
  double pAp;       // <p, A p> = ||D-hat p||^2
  double alpha;     // step length of the iteration under way
  double rho_it;    // <r, r> at its start
  double rr;        // <r, r> at its end (k_cg_end)
  double b2;        // ||b||^2
  double stop2;     // tol^2 ||b||^2 (recursive-residual target)
  double rmax;      // largest ||r|| since the last reliable update (mixed mode)
  int active;       // 1 while iterating
  int act_it;       // active at the start of the iteration under way, and no breakdown in it
  int iters;
  int status;       // wdirac_status
  int need_update;  // residual replacement requested (mixed mode: reliable update)
  int pad;
};

// Multi-shift CG (see blas.hip for the recurrences).  One system (one rhs of
// a single lattice); shift k's fields are `fstride` complex elements apart.
constexpr int MAXSHIFT = 32;
// Most iterations whose updates of x_k and p_k (k not the base shift) are applied
// together, from as many residuals kept in a ring.
constexpr int MSRING = 8;
struct ShiftList {
  double v[MAXSHIFT];
};
struct MsScalars {
  CgScalars cg;       // base recursion (rho, pAp, alpha, active, act_it, iters, status; the rest unused)
  double alpha_old, beta_old;
  double sigma0;      // base (smallest) shift
  int nshift, base;
  int xb_it;          // the base shift's x is due in the iteration under way
  int pad;
  double delta[MAXSHIFT];   // sigma_k - sigma0
  double zeta[MAXSHIFT], zeta_old[MAXSHIFT], zeta_new[MAXSHIFT];
  int sact[MAXSHIFT];     // shift k is still updated
  int siters[MAXSHIFT];   // iterations that updated shift k
  // per ring slot: x_k += as p_k where upd & 1, then p_k = zr r + bs p_k where upd & 2
  double as[MSRING][MAXSHIFT], zr[MSRING][MAXSHIFT], bs[MSRING][MAXSHIFT];
  int upd[MSRING][MAXSHIFT];
};

// Arguments of one hopping-term launch.  Pointers are device memory; fields
// are packed half spinors, links the packed represented field.
struct HopArgs {
  void *out;
  const void *in;
  const void *links;
  const void *flinks; // compact fundamental links (HOP_COMPACT forms), boundary phase folded as sqrt(bc)
  const void *xadd;   // nullable
  int nlat;
  LatDesc lat[MAXLAT];
  int parity;         // parity of the output sites
  int xcd_remap;      // map consecutive tiles to one XCD
  double alpha, beta; // out = alpha * xadd + beta * H in
  double *partial;    // nullable: per-tile partial sums of |out|^2, [system][prow]
  int prow;           // row length of `partial` (set by the launcher: the largest tile count)
  int ntiles, ngroups;  // total tiles and rhs groups (set by the launcher)
  int tblock;           // t-blocked tile order (0 = lexicographic; single lattices only), see hop.hip
  int tiles_per_tx;     // set by the launcher
  // CG iterations.  lead > 0: the first `lead` blocks (one per system) do the
  // alpha step (of the multi-shift recursion where ms is set) from the partial
  // sums lp (rows of lprow, lcnt valid) while the others hop.  lp2 (ms only):
  // lcnt2 partial sums of |p|^2.
  CgScalars *sc;
  MsScalars *ms;
  int lead, lprow, lcnt2;
  const double *lp, *lp2;
  Counts lcnt;
  // r (nullable): instead of storing out, r = rin - alpha (out + sigma ps),
  // alpha that of sc for active systems (others: r = rin), or 1 where sc is
  // NULL; `partial` then receives the sums of |r|^2.  ps is nullable, r may
  // be rin.
  void *r;
  const void *rin, *ps;
  double sigma;
  // clover block of the epilogue (hop_clover.hip): packed blocks of both
  // parities, and the field D_ee multiplies (NULL: the hop's result instead)
  const void *clov, *cx;
};

// nr: right-hand sides per block of the colour-split form (1..4; reduced to
// one that divides nrhs and fits LDS); of the site-parallel form 1 or 4 (4 rhs
// across the lanes of each wavefront).  On return counts->n[s] holds the
// number of partial sums written for system s (the tiles of its lattice) and
// *prow their row length.
hipError_t launch_hop(const HopArgs &a, int N, int rep, int d, int real, int prec, int dagger, int nrhs, int variant,
                      int nr, hipStream_t st, Counts *counts, int *prow);
// Whether the colour-split form of the given variant takes nr right-hand
// sides per block (nr in 1..4, or 6 for the unpaired form with d_R <= 4)
// within the LDS budget.
bool hop_nr_supported(int N, int d, int prec, int variant, int nr);
bool hop_variant_ok(int N, int rep, int d, int variant);
// hop_clover.hip: a hop of one right-hand side with the clover block of its
// output sites, xadd and alpha unused (complex links, d_R = 2, 3, 4, the colour
// forms of stored links).
bool hop_clover_ok(int d, int variant);
hipError_t launch_hop_clover(const HopArgs &a, int d, int prec, int dagger, int variant, hipStream_t st,
                             Counts *counts, int *prow);
// hop_mr.hip: the HOP_MULTI form (nr = right-hand sides per block, one of
// 1, 2, 3, 4, 6, 12, dividing nrhs); built for complex d_R = 3, 6 and real
// d_R = 3.
bool hop_mr_ok(int d, int real);
hipError_t launch_hop_mr(const HopArgs &a, int d, int real, int prec, int dagger, int nrhs, int nr, hipStream_t st,
                         Counts *counts, int *prow);
// Whether the compact forms exist for (N, rep): SYM for N = 2, 3, 4 and 2AS
// for N = 4 (where they read fewer bytes than the represented links).
bool compact_links_ok(int N, int rep);

// rep.hip (one lattice per call; the caller offsets the pointers)
// F (nullable): also write the compact fundamental links [parity][mu][N*N][stride]
// complex, multiplied by i where the boundary phase is -1 (the two-index maps
// are quadratic, so R(i U) = -R(U)).
hipError_t launch_rep_links(const void *U, void *UR, void *F, const Geom &g, int N, int rep, int prec,
                            hipStream_t st);
hipError_t launch_unpack_links(void *canon, const void *UR, const Geom &g, int d, int real, int prec,
                               hipStream_t st);
hipError_t launch_pack_spinor(void *packed, const void *canon, const Geom &g, int d, int parity, int nrhs,
                              int prec, int unpack, hipStream_t st);

// blas.hip -- packed half-spinor linear algebra and reductions.
struct FieldShape {
  int nsys, ncomp, maxvh;
  int vh[MAXSYS];          // sites of the system
  int stride[MAXSYS];      // padded length of one component row
  long long off[MAXSYS];   // complex elements from the field start to the system's first row
};
int blas_nblocks(const FieldShape &f);   // blocks per system of the streaming kernels (row length of partials)
Counts uniform_counts(int n);
// out = a * x + b * y (y nullable); precision of all three = prec
hipError_t launch_lincomb(void *out, double a, const void *x, double b, const void *y, const FieldShape &f, int prec,
                          hipStream_t st);
// partial[s][blk] = sum |v|^2 over the block's sites, all components
hipError_t launch_norm2_partial(double *partial, const void *v, const FieldShape &f, int prec, hipStream_t st);
// out[r] = compensated sum of partial[r][0..counts.n[r % nsys]) for r < nrows,
// rows of length prow (nrows = 2 nsys for the real and imaginary rows of a dot)
hipError_t launch_finalize_sum(double *out, const double *partial, int prow, const Counts &counts, int nrows,
                               int nsys, hipStream_t st);
// partial[s][blk] = Re sum conj(a) b, partial[nsys + s][blk] = Im sum conj(a) b
hipError_t launch_dot_partial(double *partial, const void *a, const void *b, const FieldShape &f, int prec,
                              hipStream_t st);
// out = gamma_5 x + i c y (y nullable); out may alias x or y
hipError_t launch_gamma5_axpy(void *out, const void *x, double c, const void *y, const FieldShape &f, int prec,
                              hipStream_t st);
// convert between precisions: out (prec_out) = in (prec_in)
hipError_t launch_convert(void *out, int prec_out, const void *in, int prec_in, const FieldShape &f,
                          hipStream_t st);

// CG: x += alpha p and p = r + beta p, beta from the partial sums of |r|^2
// (rows of prow); x, p, r in prec.  Also the state update of the iteration.
hipError_t launch_cg_update_xp(void *x, void *p, const void *r, CgScalars *s, const double *rr_partial, int prow,
                               const Counts &counts, double delta, const FieldShape &f, int prec, hipStream_t st);
// cg_tiny.hip: up to nit iterations of every system of a small single lattice
// (Vh d_R sites and colours in one workgroup) in one launch, until a system
// stops; x, p, r packed even fields, one block per rhs.
bool cg_tiny_ok(const Geom &g, int d, int real);
hipError_t launch_cg_tiny(void *x, void *p, void *r, const void *links, const Geom &g, int d, int real, CgScalars *s,
                          double m4, double delta, int nit, int nrhs, int prec, hipStream_t st);
// With set_b2: b2 = sum(partial), stop2 = tol^2 b2, counters reset.  Otherwise
// rho = sum(partial) for a freshly computed FP64 residual, and every system
// that is neither converged nor broken down is (re)activated.
hipError_t launch_cg_restart(CgScalars *s, const double *partial, int prow, const Counts &counts, int nsys, double tol,
                             int set_b2, hipStream_t st);
// x64 += x32, then x32 = 0
hipError_t launch_accum_x(void *x64, void *x32, const FieldShape &f, hipStream_t st);

hipError_t launch_ms_init(MsScalars *s, const double *b2_partial, int nblk, const ShiftList &delta, int nshift,
                          int base, double sigma0, double tol, hipStream_t st);
// Base shift of an iteration: x += alpha p, p = r + beta p, and the scalars
// of every shift for ring slot `slot`, beta from the partial sums of |r|^2
// (cnt of them).  pp (nullable): receives ms_base_blocks() partial sums of the
// new |p|^2.
int ms_base_blocks(const FieldShape &f);
hipError_t launch_ms_update_base(void *x, void *p, const void *r, MsScalars *s, const double *rr_partial, int cnt,
                                 int slot, double *pp, const FieldShape &f, hipStream_t st);
// The updates of the other shifts for the n iterations of ring slots 0..n-1
// (residuals `ring`, n fields fstride apart).
hipError_t launch_ms_update_xp(void *x, void *p, const void *ring, const MsScalars *s, long long fstride,
                               const FieldShape &f, int n, hipStream_t st);

// clover.hip (one lattice per call; the caller offsets the pointers).
// Clover field: [parity][chirality block][d(2d+1)][stride] complex, the upper
// triangle (row-major, diagonal included) of the Hermitian 2d x 2d block; even
// sites holding D_ee, odd sites D_oo^{-1}.  F: scratch of 6 d^2 complex FP64
// per site; Us: scratch of 4 N^2 complex FP64 per site (a structure-of-arrays
// copy of the links).
bool clover_supported(int d);
hipError_t launch_clover_field(void *clov, const void *U, double *F, double *Us, const Geom &g, int N, int rep, int d,
                               double m0, double csw, int expo, int prec, hipStream_t st);
// out = D_ee in (parity 0) or D_oo^{-1} in (parity 1); out may alias in
hipError_t launch_clover_apply(void *out, const void *in, const void *clov, const Geom &g, int d, int parity,
                               int nrhs, int prec, hipStream_t st);
// Clover contribution to the link force of a functional with variation
// -2 Re sum_x tr[dM Omega], Omega = X Y^+ (Xe non-null) or cdet D_oo^{-1} on odd
// sites (Xe NULL); P (+)= coef * force (or its gradient form).  Scratch of V
// sites: F, 6 d^2 complex FP64 (exponential form only); K, 6 d^2 reals; Gl, 24 N^2
// reals (not FUND); Us, 4 N^2 complex FP64 (structure-of-arrays links).
hipError_t launch_clover_force(void *P, const void *Xe, const void *Xo, const void *Ye, const void *Yo, const void *U,
                               const void *clov, double *F, double *K, double *Gl, double *Us, const Geom &g, int N, int rep,
                               double m0, double csw, int expo, double cdet, double coef, int gradient, int accumulate,
                               hipStream_t st);
// Partial sums of log|det D_oo(x)| over the odd sites (clover_logdet_blocks of them).
int clover_logdet_blocks(const Geom &g);
hipError_t launch_clover_logdet(const void *clov, double *partial, const Geom &g, int d, hipStream_t st);

// hmc.hip (one lattice per call; canonical fundamental links and momenta)
hipError_t launch_gauge_force(const void *U, void *F, const Geom &g, int N, double beta, double scale,
                              int accumulate, hipStream_t st);
int plaquette_blocks(const Geom &g);
hipError_t launch_plaquette_partial(const void *U, double *partial, const Geom &g, int N, hipStream_t st);
hipError_t launch_link_update(void *U, const void *pi, const Geom &g, int N, double eps, hipStream_t st);
int kinetic_blocks(const Geom &g);
hipError_t launch_kinetic_partial(const void *pi, double *partial, const Geom &g, int N, hipStream_t st);
hipError_t launch_algebra(void *pi, const double *w, const Geom &g, int N, hipStream_t st);

// force.hip (one lattice per call; the caller offsets the pointers)
// U nullable: if given, the output is 2i P U instead of P
hipError_t launch_force_links(void *P, const void *X_e, const void *X_o, const void *Y_e, const void *Y_o,
                              const void *UR, const void *U, const Geom &g, int N, int rep, double scale,
                              int accumulate, hipStream_t st);

}  // namespace wd
