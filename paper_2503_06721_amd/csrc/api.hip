// C ABI of libwdirac: argument checking, dispatch to the kernels, and the
// host loop of the conjugate-gradient solver.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/wdirac.h"
#include "wd_common.h"
#include "wd_kernels.h"

constexpr int kAuto = -1000;

struct wdirac_tuned {
  int valid, variant, nr, xcd_remap, tblock;
};

struct wdirac_ctx {
  int N, rep, d, real;
  int nlat;                        // lattices of a batch (1 for a single lattice)
  wd::Geom g[wd::MAXLAT];
  long long spre[wd::MAXLAT + 1];  // prefix sums of the packed row strides (sites)
  long long vpre[wd::MAXLAT + 1];  // prefix sums of the lattice volumes (canonical sites)
  // hop launch shape options; kAuto where the caller has set none (auto_shape)
  int hop_variant[2];   // per precision (F64, F32): one of the wd::HOP_* forms
  int hop_nr[2];        // preferred right-hand sides per colour-split block
  wdirac_tuned tuned[2][13];   // autotuned shape per (precision, nrhs)
  int xcd_remap;
  int tblock;           // t-blocked tile order (0 = lexicographic)
  int cg_check_every;   // CG iterations between host convergence checks (kAuto: check_every)
  double mixed_delta;   // reliable-update trigger ||r|| < delta max||r||
  int cg_graph;         // replay the CG iterations between checks as a HIP graph
  int tune_compact;     // the autotuner also times the compact-link forms
  mutable hipStream_t own = nullptr;   // the library's stream for graph capture (created on first use)
};

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
  g_err = msg;
  return code;
}

#define WD_HIP(expr)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) return fail(WDIRAC_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

#define WD_TRY(expr)            \
  do {                          \
    int rc_ = (expr);           \
    if (rc_ != WDIRAC_OK) return rc_; \
  } while (0)

int rep_dim(int N, int rep) {
  switch (rep) {
    case WDIRAC_FUND: return N;
    case WDIRAC_ADJ: return N * N - 1;
    case WDIRAC_SYM: return N * (N + 1) / 2;
    case WDIRAC_ASYM: return N * (N - 1) / 2;
  }
  return 0;
}

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

size_t half_bytes(const wdirac_ctx *c, int nrhs, int prec) {
  return (size_t)nrhs * 4 * c->d * c->spre[c->nlat] * (prec == WDIRAC_F64 ? 16 : 8);
}

// CG iterations between host checks: the caller's, or 4; 512 where one kernel
// runs them all and stops by itself (SU(2) FUND 4^4: an iteration 7.5 us, a check
// between kernels 21).
int check_every(const wdirac_ctx *c, bool one_kernel) {
  return c->cg_check_every != kAuto ? c->cg_check_every : one_kernel ? 512 : 4;
}

// Independent systems of a packed field: the right-hand sides of a single
// lattice, or the lattices of a batch (one right-hand side each).
int nsys_of(const wdirac_ctx *c, int nrhs) { return c->nlat == 1 ? nrhs : c->nlat; }

wd::FieldShape shape(const wdirac_ctx *c, int nrhs) {
  wd::FieldShape f{};
  f.ncomp = 4 * c->d;
  f.nsys = nsys_of(c, nrhs);
  f.maxvh = 0;
  for (int s = 0; s < f.nsys; ++s) {
    const int l = c->nlat == 1 ? 0 : s;
    f.vh[s] = c->g[l].Vh;
    f.stride[s] = c->g[l].stride;
    f.off[s] = c->nlat == 1 ? (long long)s * f.ncomp * c->g[0].stride : (long long)f.ncomp * c->spre[l];
    f.maxvh = std::max(f.maxvh, f.vh[s]);
  }
  return f;
}

hipStream_t S(void *s) { return static_cast<hipStream_t>(s); }

int check_ctx(const wdirac_ctx *c) {
  if (!c) return fail(WDIRAC_EINVAL, "ctx is NULL");
  return WDIRAC_OK;
}
int check_prec(int prec) {
  if (prec != WDIRAC_F64 && prec != WDIRAC_F32) return fail(WDIRAC_EINVAL, "prec must be WDIRAC_F64 or WDIRAC_F32");
  return WDIRAC_OK;
}
int check_nrhs(int nrhs) {
  if (nrhs < 1 || nrhs > 12) return fail(WDIRAC_EINVAL, "nrhs must be in [1, 12]");
  return WDIRAC_OK;
}
int check_nrhs(const wdirac_ctx *c, int nrhs) {
  WD_TRY(check_nrhs(nrhs));
  if (c->nlat > 1 && nrhs != 1) return fail(WDIRAC_EINVAL, "a batch of lattices carries one right-hand side");
  return WDIRAC_OK;
}
int check_parity(int p) {
  if (p != 0 && p != 1) return fail(WDIRAC_EINVAL, "parity must be 0 (even) or 1 (odd)");
  return WDIRAC_OK;
}
int check_ptr(const void *p, const char *name) {
  if (!p) return fail(WDIRAC_EINVAL, std::string(name) + " is NULL");
  return WDIRAC_OK;
}

// Workspace carving: consecutive 256-byte aligned pieces.
struct Carver {
  char *base;
  size_t off = 0;
  void *take(size_t n) {
    void *p = base ? base + off : nullptr;
    off += align256(n);
    return p;
  }
};

size_t partial_doubles(const wdirac_ctx *c, int nrhs) {
  // rows (one per system, twice for the real and imaginary rows of a dot) of
  // the longest row that hops, norms and dots write: the smallest tiles are the
  // 32-site tiles of the multi-rhs hop with two lanes per site.  (|p|^2 of the
  // multi-shift recursion has a row of its own: carve_ms.)
  int mx = 0;
  for (int l = 0; l < c->nlat; ++l) mx = std::max(mx, (c->g[l].Vh + 31) / 32);
  return (size_t)2 * nsys_of(c, nrhs) * mx;
}

struct CgWork {
  void *r, *p, *q, *t, *u, *v;            // FP64
  void *r32, *p32, *x32, *q32, *t32, *u32, *v32;  // FP32 (mixed)
  double *P1, *P2;
  wd::CgScalars *sc;
  size_t bytes;
};

CgWork carve_cg(const wdirac_ctx *c, int nrhs, int mode, void *ws) {
  Carver cv{static_cast<char *>(ws)};
  CgWork w{};
  const size_t h64 = half_bytes(c, nrhs, WDIRAC_F64), h32 = half_bytes(c, nrhs, WDIRAC_F32);
  w.r = cv.take(h64); w.p = cv.take(h64); w.q = cv.take(h64);
  w.t = cv.take(h64); w.u = cv.take(h64); w.v = cv.take(h64);
  if (mode == WDIRAC_CG_MIXED) {
    w.r32 = cv.take(h32); w.p32 = cv.take(h32); w.x32 = cv.take(h32); w.q32 = cv.take(h32);
    w.t32 = cv.take(h32); w.u32 = cv.take(h32); w.v32 = cv.take(h32);
  }
  w.P1 = static_cast<double *>(cv.take(partial_doubles(c, nrhs) * sizeof(double)));
  w.P2 = static_cast<double *>(cv.take(partial_doubles(c, nrhs) * sizeof(double)));
  w.sc = static_cast<wd::CgScalars *>(cv.take(nsys_of(c, nrhs) * sizeof(wd::CgScalars)));
  w.bytes = cv.off;
  return w;
}

// Residuals that a multi-shift solve keeps.  Each costs a half field of workspace
// and defers the updates of the nshift - 1 other shifts, so few shifts keep few
// (SU(3) FUND 32^4, us an iteration with 3, this many and 8 residuals: 2 shifts
// 810, 810, 793; 4 shifts 886, 858, 839; 12 shifts 1220, 1036, 1036).  Two shifts
// then need 7 half fields, no more than with an update in every iteration.
int ms_ring(int nshift) { return nshift == 1 ? 1 : std::min(wd::MSRING, nshift + 1); }

struct MsWork {
  void *r, *t, *u, *p;       // FP64 half fields; r holds a ring of residuals, p nshift fields
  int ring;                  // residuals kept: one where only the base shift needs them
  double *P1, *P2, *P3;
  wd::MsScalars *sc;
  size_t bytes;
};

MsWork carve_ms(const wdirac_ctx *c, int nshift, void *ws) {
  Carver cv{static_cast<char *>(ws)};
  MsWork w{};
  const size_t h = half_bytes(c, 1, WDIRAC_F64);
  w.ring = ms_ring(nshift);
  w.r = cv.take((size_t)w.ring * h);
  w.t = cv.take(h); w.u = cv.take(h);
  w.p = cv.take((size_t)nshift * h);
  w.P1 = static_cast<double *>(cv.take(partial_doubles(c, 1) * sizeof(double)));
  w.P2 = static_cast<double *>(cv.take(partial_doubles(c, 1) * sizeof(double)));
  w.P3 = static_cast<double *>(cv.take(wd::ms_base_blocks(shape(c, 1)) * sizeof(double)));
  w.sc = static_cast<wd::MsScalars *>(cv.take(sizeof(wd::MsScalars)));
  w.bytes = cv.off;
  return w;
}

// Bytes of the represented links of the whole context in precision prec; the
// compact fundamental copy (two-index representations with compact forms)
// follows them in the same links field.
size_t rep_links_bytes(const wdirac_ctx *c, int prec) {
  return (size_t)8 * c->d * c->d * c->spre[c->nlat] * (prec == WDIRAC_F64 ? 8 : 4) * (c->real ? 1 : 2);
}
size_t compact_links_bytes(const wdirac_ctx *c, int prec) {
  if (!wd::compact_links_ok(c->N, c->rep)) return 0;
  return (size_t)8 * c->N * c->N * c->spre[c->nlat] * (prec == WDIRAC_F64 ? 16 : 8);
}

// Right-hand sides per colour-split block: the largest supported divisor of
// nrhs not above the preference.
int effective_nr(const wdirac_ctx *c, int pref, int nrhs, int prec, int variant) {
  // site-parallel form: 4 right-hand sides across the lanes of a wavefront, or 1
  if (variant == wd::HOP_SITE) return (pref >= 4 && nrhs % 4 == 0) ? 4 : 1;
  for (int nr = std::min(pref, variant == wd::HOP_MULTI ? 12 : 6); nr > 1; --nr)
    if (nrhs % nr == 0 && wd::hop_nr_supported(c->N, c->d, prec, variant, nr)) return nr;
  return 1;
}

// Whether the 32-bit offsets of the multi-rhs form reach the whole lattice
// (its largest: an entry of a (parity, direction) block of links, 16 bytes).
bool hop_mr_reaches(const wdirac_ctx *c) {
  for (int l = 0; l < c->nlat; ++l)
    if ((long long)c->d * c->d * c->g[l].stride * 16 >= 1ll << 32) return false;
  return true;
}

// Launch shape of a hop the caller has neither tuned nor set options for, by
// representation, precision, right-hand sides and size (half-lattice sites
// Vh).  Times are us per hop, the shape chosen against the one across the line;
// where none is named, that is the colour-split form with one hop per phase and
// up to four rhs per block.
//  * Two-index links, FP64: the compact form reads N^2 instead of d_R^2
//    entries per link and rebuilds the others by the formula of rep_links from
//    the same links (SU(3) SYM 24^4: 92 against 178, SU(4) 2AS 130 against 179,
//    SU(4) SYM 188 against 397; 2AS below 16^4 is faster with stored links).
//    Not in FP32, where entries rebuilt from rounded links carry a larger error.
//    d_R = 10 takes two rhs per block as soon as one would leave a CU with two
//    blocks (SU(4) SYM 8^4, 10 rhs: 26 against 32 with one; 8 rhs, 256 blocks:
//    18 with one against 26).
//  * Several rhs at d_R = 6: one wavefront per rhs with the links staged per
//    block, swept along t over sub-lattices so that neighbours stay in L2
//    (SU(3) SYM 48x24^3, 12 rhs FP64: 1454 against 2004, FP32 836 against
//    988).
//    - SYM in FP64 is faster one rhs per block in the compact form below six
//      rhs (24^4, 4 rhs: 303 against 350) and where no sweep fits (18x14^3, 8
//      rhs: 85 against 88), but for lattices whose compact blocks, three per CU,
//      take a second round and whose fields still fit the caches (10^4, 12 rhs:
//      26 against 35; 12^4, 8 rhs: 37 against 44; level at 14^4, 12 rhs: 98).
//    - FP32 with two or three rhs only on large lattices (24^4, 2 rhs: 113
//      against 123 for two hops per phase; 20^4: 62 against 52).
//    - Four, three or two rhs per block, the most that divide nrhs; in FP32 two
//      on lattices too small for the blocks that larger groups leave, the fewer
//      the groups the larger (four against two: 4 rhs 32x16^3 74 against 62,
//      20^4 87 either way, 24^4 163 against 183; 8 rhs 10^4 15.5 against 15.0,
//      12^4 21.7 against 23.6; 12 rhs 8^4 12.7 against 12.6, 10x14x6x18 22 against
//      25; three against two: 6 rhs 12^4 17.9 against 17.2, 16x8x12x16 18.0
//      against 20.2).
//    - Sub-lattices of three x-rows by three tiles, else four (24^4, 12 rhs FP32:
//      422 against 434 for four by three); a row of four tiles by two in FP64
//      (32x16^3, 12 rhs: 299 against 309; 24x16^3 217 against 219; 16^4 186 against
//      174), by four in FP32 (24x16^3, 8 rhs: 71 against 75).  With fewer than six
//      rhs only by three tiles (24^4, 4 rhs FP32: 163 against 173 without a sweep;
//      32x16^3, rows of four tiles: 97 against 62).
//  * d_R <= 4, one rhs: two or four hops per phase, more loads in flight per
//    barrier (SU(3) FUND 32^4 FP64: 135 against 155, FP32 79 against 86; 24^4:
//    51.5 against 53.4; SU(2) FUND 16^4 7.8 against 9.0).
//  * d_R <= 4, several rhs in FP64: two hops per phase with two or three rhs per
//    block (24^4, 12 rhs: SU(3) FUND 389 against 476, SU(2) ADJ 326 against
//    440).  d_R = 4 gains with 2 or 4 rhs (24^4, 4 rhs: 196 against 204), two rhs
//    in blocks of one below 20000 sites (8^4: 7.2 against 8.7; 14^4: 15.3 against
//    16.4; 24^4: 121 against 114); with others where groups of four fill the
//    chip poorly (16^4, 12 rhs: 93 against 107; 24^4: 556 against 534; 12^4: 31
//    against 29; groups of three, 6 rhs: 16^4 51 against 54, 16^3x8 25.5 against
//    24.0).  SU(2) SYM with 5, 7 or 11 rhs takes stored links on small lattices
//    (10^4, 5 rhs: 8.0 against 9.1; 10x14x6x18 10.4 against 10.5, 7 rhs 12.7
//    against 12.4).
//  * d_R = 15: fewer rhs per block, four spill (SU(4) ADJ 24^4 FP32, 12 rhs:
//    1788 against 3083).
//  * XCD ranges are left out where each would start a multiple of 128 KiB into
//    every row and the fields outgrow the memory-side cache: the eight XCDs then
//    stream the same HBM channels at the same time (SU(3) FUND 32^4 FP64 135
//    against 147 with ranges, FP32 79 against 87; 24x32^3: 103 against 115, FP32
//    62 against 64; 36x32^3, a multiple in FP64 alone: 168 against 175, FP32 99
//    against 93; 24^4, whose ranges do not line up: 51.6 either way; 16^4, in
//    cache: 12.6 against 11.5), and for the stored links of d_R = 6, which
//    nothing re-reads (SU(4) 2AS 48x24^3 FP32: 178 against 185).
wdirac_tuned auto_shape(const wdirac_ctx *c, int prec, int nrhs) {
  const bool f64 = prec == WDIRAC_F64, even = nrhs % 2 == 0;
  long long Vh = 0, tiles = 0;   // tiles of 64 sites
  for (int l = 0; l < c->nlat; ++l) {
    Vh += c->g[l].Vh;
    tiles += (c->g[l].Vh + 63) / 64;
  }
  const bool large = Vh >= 131072;
  const bool odd = nrhs > 3 && nrhs % 2 && nrhs % 3;   // 5, 7, 11: one rhs per block in every form
  const int d = c->d;
  wdirac_tuned s{1, wd::HOP_COLOUR, 4, 1, 0};
  if (d == 6) {
    // sweep of bx x-rows by by tiles of 32 sites of a (t, x) row
    const wd::Geom &g = c->g[0];
    const int nb = g.Y * g.Z % 64 == 0 ? g.Y * g.Z / 64 : 0;
    const int bx = g.X % 3 == 0 ? 3 : g.X % 4 == 0 ? 4 : 2;
    const int by = nb == 0 ? 0 : nb % 3 == 0 ? 3 : nb % 4 == 0 && (nb >= 8 || !f64) ? 4 : nb % 2 == 0 ? 2 : 0;
    const bool sym = c->rep == WDIRAC_SYM;
    const bool pairs = !f64 && even && Vh < (nrhs < 6 ? 75000 : nrhs < 8 ? 12288 : nrhs < 12 ? 6000 : 4096);
    const int nr = pairs ? 2 : nrhs % 4 == 0 ? 4 : nrhs % 3 == 0 ? 3 : even ? 2 : 1;
    const bool rounds = Vh < 16384 && tiles * nrhs > 768;   // of the compact form's blocks
    const bool multi = nr > 1 && hop_mr_reaches(c) &&
                       (!f64 ? large || nrhs >= 4 : sym ? nrhs >= 6 && (by > 0 || rounds) : nrhs >= 3);
    if (multi) {
      s.variant = wd::HOP_MULTI;
      s.nr = nr;
      s.tblock = by == 3 || (by && nrhs >= 6) ? -(10 * bx + by) : 0;
    } else if (f64 && (sym || (nrhs == 1 && Vh >= 16384) || (nrhs == 2 && Vh >= 32768))) {
      s.variant = wd::HOP_COMPACT;
      s.nr = sym ? 1 : nrhs;
    } else if (nrhs == 1 || (f64 && nrhs > 2)) {
      s.variant = wd::HOP_COLOUR_PAIR;
      s.nr = f64 && even ? 2 : 1;
      if (!f64 && large && c->nlat == 1) s.xcd_remap = 0;
    }
  } else if (f64 && wd::compact_links_ok(c->N, c->rep) && !(d == 3 && odd && Vh < 7000)) {   // SYM, d_R = 3 and 10
    s.variant = wd::HOP_COMPACT;
    s.nr = d == 10 && even && tiles * nrhs > 256 ? 2 : 1;
  } else if (d <= 4 && nrhs == 1) {
    s.variant = f64 ? (d == 2 && !large ? wd::HOP_COLOUR_PAIR : wd::HOP_COLOUR_QUAD)
                    : (d == 3 && !c->real ? wd::HOP_COLOUR_PAIR : wd::HOP_COLOUR_QUAD);
  } else if (f64 && (d == 2 || d == 3 || (d == 4 && (nrhs == 2 || nrhs == 4 || (!large && (nrhs < 6 || Vh >= (nrhs % 4 ? 20000 : 16384))))))) {
    const bool two = nrhs > 2 || (d == 4 ? Vh >= 20000 : d == 3 && !c->real);   // rhs per block, if even
    s.variant = wd::HOP_COLOUR_PAIR;
    s.nr = d == 3 && nrhs % 3 == 0 && Vh >= 65536 ? 3 : even && two ? 2 : 1;
  } else if (d == 2 && even && Vh < 262144) {               // FP32
    s.nr = 2;
  } else if (d == 15) {
    s.nr = f64 ? 1 : even ? 2 : 4;
  } else if (nrhs == 1 || (f64 && (nrhs == 2 || nrhs == 4))) {   // ADJ d_R = 8; SYM d_R = 10 in FP32
    s.variant = wd::HOP_COLOUR_PAIR;
    s.nr = 1;
  }
  // (one rhs only: the rhs groups of a tile share its links in one XCD's L2)
  if (c->nlat == 1 && nrhs == 1 && Vh >= 262144 && Vh % (f64 ? 65536 : 131072) == 0 && (f64 || d < 15)) s.xcd_remap = 0;
  return s;
}

// What a hop of a CG iteration does beside hopping (wd_kernels.h, HopArgs):
// the alpha step from the partial sums lp, or the update of the residual r.
struct CgHop {
  wd::CgScalars *sc = nullptr;
  int lead = 0;         // leading blocks of the alpha step (0: none)
  const double *lp = nullptr;
  int lprow = 0;
  wd::Counts lcnt{};
  void *r = nullptr;    // r = rin - alpha (A p + sigma ps)
  const void *rin = nullptr, *ps = nullptr;
  double sigma = 0.0;
  wd::MsScalars *ms = nullptr;
  const double *lp2 = nullptr;
  int lcnt2 = 0;
};

// D_ee in (parity 0) or D_oo^{-1} in (parity 1) with a clover field, lattice
// by lattice; out may alias in.
int clover_apply(const wdirac_ctx *c, void *out, const void *in, const void *clov, int parity, int nrhs, int prec,
                 hipStream_t st) {
  const size_t cb = prec == WDIRAC_F64 ? 16 : 8;
  for (int l = 0; l < c->nlat; ++l) {
    const size_t so = (size_t)4 * c->d * c->spre[l] * cb;
    const size_t co = (size_t)4 * c->d * (2 * c->d + 1) * c->spre[l] * cb;
    WD_HIP(wd::launch_clover_apply(static_cast<char *>(out) + so, static_cast<const char *>(in) + so,
                                   static_cast<const char *>(clov) + co, c->g[l], c->d, parity, nrhs, prec, st));
  }
  return WDIRAC_OK;
}

// One hopping-term launch over every lattice of the context.  counts/prow
// (nullable) receive the layout of the per-tile partial sums.
// clov (nullable): out = D_oo^{-1} (beta H in) on the odd sites, out = D_ee cx +
// beta H in on the even ones (alpha and xadd unused), in the hop's epilogue where
// one of its forms is launched, else by a pass of its own.
int hop(const wdirac_ctx *c, void *out, const void *in, const void *UR, int out_parity, int dagger, int nrhs,
        double alpha, const void *xadd, double beta, int prec, double *partial, hipStream_t st,
        wd::Counts *counts = nullptr, int *prow = nullptr, const CgHop *cg = nullptr, const void *clov = nullptr,
        const void *cx = nullptr) {
  wdirac_tuned sh = c->tuned[prec][nrhs];
  if (!sh.valid) {
    sh = auto_shape(c, prec, nrhs);
    if (c->hop_variant[prec] != kAuto) sh = wdirac_tuned{1, c->hop_variant[prec], 4, 1, 0};
    if (c->hop_nr[prec] != kAuto) sh.nr = c->hop_nr[prec];
    if (c->xcd_remap != kAuto) sh.xcd_remap = c->xcd_remap;
    if (c->tblock != kAuto) sh.tblock = c->tblock;
  }
  // (the multi-rhs form loads whole 16-byte link entries directly into LDS)
  if (sh.variant == wd::HOP_MULTI && (!hop_mr_reaches(c) || ((size_t)UR & 15))) sh.variant = wd::HOP_COLOUR;
  const bool fused = clov && nrhs == 1 && !c->real && wd::hop_clover_ok(c->d, sh.variant);
  if (clov && cx && !fused) {
    WD_TRY(clover_apply(c, out, cx, clov, 0, nrhs, prec, st));
    xadd = out;
    alpha = 1.0;
  }
  wd::HopArgs a;
  a.clov = clov;
  a.cx = cx;
  a.out = out;
  a.in = in;
  a.links = UR;
  a.flinks = wd::compact_links_ok(c->N, c->rep) ? static_cast<const char *>(UR) + rep_links_bytes(c, prec) : nullptr;
  a.xadd = xadd;
  a.nlat = c->nlat;
  for (int l = 0; l < c->nlat; ++l) {
    a.lat[l].g = c->g[l];
    a.lat[l].tile0 = a.lat[l].ntiles = 0;
    a.lat[l].soff = c->nlat == 1 ? 0 : (long long)4 * c->d * c->spre[l];
    a.lat[l].loff = (long long)8 * c->d * c->d * c->spre[l];
    a.lat[l].floff = (long long)8 * c->N * c->N * c->spre[l];
  }
  a.parity = out_parity;
  a.xcd_remap = sh.xcd_remap;
  a.alpha = alpha;
  a.beta = beta;
  a.partial = partial;
  a.prow = a.ntiles = a.ngroups = 0;
  a.tblock = c->nlat == 1 ? sh.tblock : 0;
  a.tiles_per_tx = 0;
  const CgHop none, &h = cg ? *cg : none;
  a.sc = h.sc;
  a.ms = h.ms;
  a.lead = h.lead;
  a.lp = h.lp;
  a.lprow = h.lprow;
  a.lcnt = h.lcnt;
  a.lp2 = h.lp2;
  a.lcnt2 = h.lcnt2;
  a.r = h.r;
  a.rin = h.rin;
  a.ps = h.ps;
  a.sigma = h.sigma;
  wd::Counts cnt{};
  int pr = 0;
  if (fused)
    WD_HIP(wd::launch_hop_clover(a, c->d, prec, dagger, sh.variant, st, &cnt, &pr));
  else
    WD_HIP(wd::launch_hop(a, c->N, c->rep, c->d, c->real, prec, dagger, nrhs, sh.variant,
                          effective_nr(c, sh.nr, nrhs, prec, sh.variant), st, &cnt, &pr));
  if (clov && !cx && !fused) WD_TRY(clover_apply(c, out, out, clov, 1, nrhs, prec, st));
  if (counts) *counts = cnt;
  if (prow) *prow = pr;
  return WDIRAC_OK;
}

// out = D-hat in (dagger = 0) or D-hat^+ in (dagger = 1); tmp is an odd half field.
// Without a clover field: D-hat = (4+m)^2 - D_eo D_oe (Sec. 5.3.3, one factor
// of 4+m absorbed).  With one: D-hat = D_ee - D_eo D_oo^{-1} D_oe, whose
// diagonal blocks are Hermitian, so the adjoint only swaps to the dagger hops.
// cg1, cg2 (nullable): what the first and the second hop do for a CG iteration.
int dhat(const wdirac_ctx *c, void *out, const void *in, const void *UR, double m0, int dagger, int nrhs, int prec,
         void *tmp, double *partial, hipStream_t st, wd::Counts *counts = nullptr, int *prow = nullptr,
         const void *clov = nullptr, const CgHop *cg1 = nullptr, const CgHop *cg2 = nullptr) {
  WD_TRY(hop(c, tmp, in, UR, 1, dagger, nrhs, 0.0, nullptr, 1.0, prec, nullptr, st, nullptr, nullptr, cg1, clov));
  if (clov)
    return hop(c, out, tmp, UR, 0, dagger, nrhs, 0.0, nullptr, -1.0, prec, partial, st, counts, prow, cg2, clov, in);
  return hop(c, out, tmp, UR, 0, dagger, nrhs, (4.0 + m0) * (4.0 + m0), in, -1.0, prec, partial, st, counts, prow,
             cg2);
}

// Canonical <-> packed half spinors, lattice by lattice.  Canonical batch
// layout: [lattice][T][X][Y][Z][4][d] (one right-hand side).
int pack(const wdirac_ctx *c, void *packed, void *canon, int parity, int nrhs, int prec, int unpack, hipStream_t st) {
  const size_t cb = prec == WDIRAC_F64 ? 16 : 8;
  for (int l = 0; l < c->nlat; ++l) {
    char *P = static_cast<char *>(packed) + (size_t)4 * c->d * c->spre[l] * cb;
    char *C = static_cast<char *>(canon) + (size_t)4 * c->d * c->vpre[l] * cb;
    WD_HIP(wd::launch_pack_spinor(P, C, c->g[l], c->d, parity, nrhs, prec, unpack, st));
  }
  return WDIRAC_OK;
}

// Workspace of the clover force: the three FP64 half fields of the
// pseudofermion force (whole batch), then the per-lattice scratch of the
// largest lattice: F (6 d^2 V), K and the leaf matrices (room for 12 d^2 V and
// 24 N^2 V) complex FP64, and the log-det partial sums.
struct CloverForceWs {
  void *z_o, *y_e, *w_o;
  double *F, *K, *G, *Us, *part, *dtmp;
  size_t bytes;
};

CloverForceWs carve_clover_force(const wdirac_ctx *c, void *base) {
  Carver cv{static_cast<char *>(base)};
  CloverForceWs w;
  const size_t h = half_bytes(c, 1, WDIRAC_F64);
  w.z_o = cv.take(h);
  w.y_e = cv.take(h);
  w.w_o = cv.take(h);
  size_t V = 0;
  int nb = 0;
  for (int l = 0; l < c->nlat; ++l) {
    V = std::max(V, 2 * (size_t)c->g[l].Vh);
    nb = std::max(nb, wd::clover_logdet_blocks(c->g[l]));
  }
  const size_t d2 = (size_t)c->d * c->d, n2 = (size_t)c->N * c->N;
  w.F = static_cast<double *>(cv.take(6 * d2 * V * 16));
  w.K = static_cast<double *>(cv.take(12 * d2 * V * 16));
  w.G = static_cast<double *>(cv.take(24 * n2 * V * 16));
  w.Us = static_cast<double *>(cv.take(4 * n2 * V * 16));
  w.part = static_cast<double *>(cv.take((size_t)nb * sizeof(double)));
  w.dtmp = static_cast<double *>(cv.take(sizeof(double)));
  w.bytes = cv.off;
  return w;
}

}  // namespace

extern "C" {

const char *wdirac_last_error(void) { return g_err.c_str(); }

int wdirac_create_batch(wdirac_ctx **ctx, int Ng, int rep, const wdirac_geom *geoms, int nlat) {
  g_err.clear();
  if (!ctx) return fail(WDIRAC_EINVAL, "ctx is NULL");
  *ctx = nullptr;
  if (!geoms) return fail(WDIRAC_EINVAL, "geom is NULL");
  if (nlat < 1 || nlat > wd::MAXLAT) return fail(WDIRAC_EINVAL, "a batch holds 1 to 8 lattices");
  if (rep < WDIRAC_FUND || rep > WDIRAC_ASYM) return fail(WDIRAC_EINVAL, "unknown representation");
  if (Ng < 2 || Ng > 4) return fail(WDIRAC_EUNSUPPORTED, "Ng must be 2, 3 or 4");
  if (Ng == 2 && rep == WDIRAC_ASYM) return fail(WDIRAC_EUNSUPPORTED, "SU(2) 2AS is one-dimensional (d_R = 1)");
  const int d = rep_dim(Ng, rep);
  int64_t total = 0;
  for (int l = 0; l < nlat; ++l) {
    int64_t V = 1;
    for (int mu = 0; mu < 4; ++mu) {
      const int L = geoms[l].dims[mu];
      if (L < 2 || (L & 1)) return fail(WDIRAC_EINVAL, "every lattice extent must be even and >= 2");
      if (geoms[l].bc[mu] != 1 && geoms[l].bc[mu] != -1) return fail(WDIRAC_EINVAL, "bc must be +1 or -1");
      V *= L;
    }
    if (V > (int64_t)1 << 30) return fail(WDIRAC_EINVAL, "lattice volume above 2^30 sites");
    total += V;
  }
  // every packed offset must stay addressable by the kernels' 64-bit arithmetic
  // and every per-lattice row index by 32-bit ints (checked per lattice above)
  if (total * 12 * d * d > ((int64_t)1 << 45)) return fail(WDIRAC_EINVAL, "batch too large");
  wdirac_ctx *c = new wdirac_ctx();
  c->N = Ng;
  c->rep = rep;
  c->d = d;
  c->real = rep == WDIRAC_ADJ;
  c->nlat = nlat;
  c->spre[0] = c->vpre[0] = 0;
  for (int l = 0; l < nlat; ++l) {
    wd::Geom &g = c->g[l];
    g.T = geoms[l].dims[0];
    g.X = geoms[l].dims[1];
    g.Y = geoms[l].dims[2];
    g.Z = geoms[l].dims[3];
    const int64_t V = (int64_t)g.T * g.X * g.Y * g.Z;
    g.Vh = (int)(V / 2);
    // Rows of whole 256-site tiles (see hop.hip).  A row pitch that is a
    // multiple of 16 KB (1024 FP64 complex entries) puts the component rows
    // a wavefront streams together on the same HBM channel pattern; such
    // strides are padded by 256 entries (7-read/1-write streaming probe with
    // 256 MiB rows: 5.74 TB/s, rows 4 KB off a 16 KB multiple: 6.04 TB/s).
    g.stride = (g.Vh + 255) & ~255;
    if (g.stride % 1024 == 0) g.stride += 256;
    for (int mu = 0; mu < 4; ++mu) g.bc[mu] = geoms[l].bc[mu];
    g.dX.set(g.X);
    g.dY.set(g.Y);
    g.dZ.set(g.Z);
    c->spre[l + 1] = c->spre[l] + g.stride;
    c->vpre[l + 1] = c->vpre[l] + V;
  }
  c->hop_variant[0] = c->hop_variant[1] = c->hop_nr[0] = c->hop_nr[1] = kAuto;
  std::memset(c->tuned, 0, sizeof(c->tuned));
  c->xcd_remap = c->tblock = c->cg_check_every = kAuto;
  c->mixed_delta = 0.01;
  c->cg_graph = 1;
  c->tune_compact = 1;
  *ctx = c;
  return WDIRAC_OK;
}

int wdirac_create(wdirac_ctx **ctx, int Ng, int rep, const wdirac_geom *geom) {
  return wdirac_create_batch(ctx, Ng, rep, geom, 1);
}

int wdirac_destroy(wdirac_ctx *ctx) {
  if (ctx && ctx->own) (void)hipStreamDestroy(ctx->own);
  delete ctx;
  return WDIRAC_OK;
}

int wdirac_rep_info(const wdirac_ctx *ctx, int *d_R, int *real_links) {
  WD_TRY(check_ctx(ctx));
  if (d_R) *d_R = ctx->d;
  if (real_links) *real_links = ctx->real;
  return WDIRAC_OK;
}

size_t wdirac_field_bytes(const wdirac_ctx *ctx, int kind, int nrhs, int prec) {
  if (!ctx || (prec != WDIRAC_F64 && prec != WDIRAC_F32)) return 0;
  const size_t el = prec == WDIRAC_F64 ? 8 : 4;
  if (kind == WDIRAC_FIELD_HALF_SPINOR) {
    if (nrhs < 1 || nrhs > 12) return 0;
    return half_bytes(ctx, nrhs, prec);
  }
  if (kind == WDIRAC_FIELD_LINKS) return rep_links_bytes(ctx, prec) + compact_links_bytes(ctx, prec);
  if (kind == WDIRAC_FIELD_CLOVER)
    return wd::clover_supported(ctx->d) ? (size_t)4 * ctx->d * (2 * ctx->d + 1) * ctx->spre[ctx->nlat] * 2 * el : 0;
  return 0;
}

size_t wdirac_workspace_bytes(const wdirac_ctx *ctx, int op, int nrhs, int prec) {
  if (!ctx) return 0;
  if (op == WDIRAC_OP_GAUGE) {   // reductions over links and sites
    int mx = 0;
    for (int l = 0; l < ctx->nlat; ++l) mx = std::max(mx, wd::kinetic_blocks(ctx->g[l]));
    return align256((size_t)mx * sizeof(double)) + align256(sizeof(double));
  }
  if (op == WDIRAC_OP_CLOVER) {   // scratch of the clover-field construction
    if (!wd::clover_supported(ctx->d)) return 0;
    int mx = 0;
    for (int l = 0; l < ctx->nlat; ++l) mx = std::max(mx, ctx->g[l].Vh);
    // F, then the structure-of-arrays copy of the links
    return align256((size_t)6 * ctx->d * ctx->d * 2 * mx * 16) + align256((size_t)4 * ctx->N * ctx->N * 2 * mx * 16);
  }
  if (op == WDIRAC_OP_CLOVER_FORCE) {
    if (!wd::clover_supported(ctx->d)) return 0;
    return carve_clover_force(ctx, nullptr).bytes;
  }
  if (op == WDIRAC_OP_MSHIFT) {   // nrhs = number of shifts
    if (nrhs < 1 || nrhs > wd::MAXSHIFT || prec != WDIRAC_F64 || ctx->nlat != 1) return 0;
    return carve_ms(ctx, nrhs, nullptr).bytes;
  }
  if (nrhs < 1 || nrhs > 12 || (ctx->nlat > 1 && nrhs != 1)) return 0;
  switch (op) {
    case WDIRAC_OP_DHAT:
      if (prec != WDIRAC_F64 && prec != WDIRAC_F32) return 0;
      return align256(half_bytes(ctx, nrhs, prec));
    case WDIRAC_OP_CG:
      if (prec != WDIRAC_CG_F64 && prec != WDIRAC_CG_MIXED) return 0;
      return carve_cg(ctx, nrhs, prec, nullptr).bytes;
    case WDIRAC_OP_FORCE:
      return 3 * align256(half_bytes(ctx, 1, WDIRAC_F64));
    case WDIRAC_OP_NORM:
    case WDIRAC_OP_DOT:
      return align256(partial_doubles(ctx, nrhs) * sizeof(double)) + align256(2 * wd::MAXSYS * sizeof(double));
    case WDIRAC_OP_TUNE:
      if (prec != WDIRAC_F64 && prec != WDIRAC_F32) return 0;
      return 3 * align256(half_bytes(ctx, nrhs, prec));
  }
  return 0;
}

int wdirac_set_option(wdirac_ctx *ctx, int option, double value) {
  WD_TRY(check_ctx(ctx));
  switch (option) {
    case WDIRAC_OPT_HOP_VARIANT_F64:
    case WDIRAC_OPT_HOP_VARIANT_F32: {
      const int v = (int)value;
      if (v < wd::HOP_SITE || v > wd::HOP_MULTI) return fail(WDIRAC_EINVAL, "hop variant out of range");
      if (!wd::hop_variant_ok(ctx->N, ctx->rep, ctx->d, v))
        return fail(WDIRAC_EUNSUPPORTED, "hop variant not available for this representation");
      ctx->hop_variant[option == WDIRAC_OPT_HOP_VARIANT_F64 ? 0 : 1] = v;
      return WDIRAC_OK;
    }
    case WDIRAC_OPT_XCD_REMAP:
      ctx->xcd_remap = value != 0.0;
      return WDIRAC_OK;
    case WDIRAC_OPT_CG_CHECK_EVERY:
      if (value < 1 || value > 1000) return fail(WDIRAC_EINVAL, "check interval must be in [1, 1000]");
      ctx->cg_check_every = (int)value;
      return WDIRAC_OK;
    case WDIRAC_OPT_MIXED_DELTA:
      if (!(value > 0.0 && value < 1.0)) return fail(WDIRAC_EINVAL, "delta must be in (0, 1)");
      ctx->mixed_delta = value;
      return WDIRAC_OK;
    case WDIRAC_OPT_CG_GRAPH:
      if (value != 0.0 && value != 1.0) return fail(WDIRAC_EINVAL, "CG graph option must be 0 or 1");
      ctx->cg_graph = (int)value;
      return WDIRAC_OK;
    case WDIRAC_OPT_TILE_TBLOCK:
      if (!(value >= -99 && value <= 64)) return fail(WDIRAC_EINVAL, "t-block must be in [-99, 64]");
      ctx->tblock = (int)value;
      return WDIRAC_OK;
    case WDIRAC_OPT_TUNE_COMPACT:
      if (value != 0.0 && value != 1.0) return fail(WDIRAC_EINVAL, "compact tuning option must be 0 or 1");
      ctx->tune_compact = (int)value;
      return WDIRAC_OK;
    case WDIRAC_OPT_HOP_NR_F64:
    case WDIRAC_OPT_HOP_NR_F32:
      if (!(value >= 1 && value <= 12)) return fail(WDIRAC_EINVAL, "right-hand sides per block must be in [1, 12]");
      ctx->hop_nr[option == WDIRAC_OPT_HOP_NR_F64 ? 0 : 1] = (int)value;
      return WDIRAC_OK;
  }
  return fail(WDIRAC_EINVAL, "unknown option");
}

int wdirac_autotune(wdirac_ctx *ctx, const void *UR, int prec, int nrhs, void *workspace, wdirac_tuning *best,
                    void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_prec(prec));
  WD_TRY(check_nrhs(ctx, nrhs));
  const hipStream_t st = S(stream);
  Carver cv{static_cast<char *>(workspace)};
  const size_t hb = half_bytes(ctx, nrhs, prec);
  void *f0 = cv.take(hb), *f1 = cv.take(hb), *f2 = cv.take(hb);
  WD_HIP(hipMemsetAsync(f0, 0, hb, st));
  WD_HIP(hipMemsetAsync(f1, 0, hb, st));
  WD_HIP(hipMemsetAsync(f2, 0, hb, st));
  struct Cand {
    int variant, nr, remap, tblock;
  };
  std::vector<Cand> cands;
  // sub-lattice sweeps (negative codes -(10 bx + by)) only where a work item
  // holds several right-hand sides; shapes whose code does not fit the
  // lattice fall back to lexicographic order in the launch
  const int tbs[] = {0, 2, 4, 8, -23, -33, -43, -63, -39};
  for (int tb : tbs) {
    if (tb < 0 && nrhs < 4) continue;
    if (tb > 0 && (ctx->nlat > 1 || ctx->g[0].T % tb)) continue;
    if (tb < 0 && (ctx->nlat > 1 || ctx->g[0].X % ((-tb) / 10))) continue;
    for (int remap = 0; remap < 2; ++remap) {
      for (int v = wd::HOP_COLOUR; v <= wd::HOP_MULTI; ++v) {
        if (!wd::hop_variant_ok(ctx->N, ctx->rep, ctx->d, v)) continue;
        if (!ctx->tune_compact && (v == wd::HOP_COMPACT || v == wd::HOP_COMPACT_PAIR)) continue;
        // the multi-rhs form only where it shares links (nr > 1)
        for (int nr : {1, 2, 3, 4, 6, 12})
          if ((v != wd::HOP_MULTI || nr > 1) && effective_nr(ctx, nr, nrhs, prec, v) == nr)
            cands.push_back({v, nr, remap, tb});
      }
      if (wd::hop_variant_ok(ctx->N, ctx->rep, ctx->d, wd::HOP_SITE)) {
        cands.push_back({wd::HOP_SITE, 1, remap, tb});
        if (nrhs % 4 == 0) cands.push_back({wd::HOP_SITE, 4, remap, tb});
      }
    }
  }
  hipEvent_t e0, e1;
  WD_HIP(hipEventCreate(&e0));
  WD_HIP(hipEventCreate(&e1));
  wdirac_tuned &slot = ctx->tuned[prec][nrhs];
  int rc = WDIRAC_OK;
  // Mean time of `reps` back-to-back launches of candidate cd (after 4
  // untimed), alternating D_eo f0 -> f1 and D_oe f1 -> f2: every other
  // launch reads the output just written, as between the hops of a solver.
  auto time_cand = [&](const Cand &cd, int reps, float *ms) {
    slot = wdirac_tuned{1, cd.variant, cd.nr, cd.remap, cd.tblock};
    auto launch = [&](int k) {
      return hop(ctx, (k & 1) ? f2 : f1, (k & 1) ? f1 : f0, UR, k & 1, 0, nrhs, 0.0, nullptr, 1.0, prec, nullptr,
                 st);
    };
    for (int k = 0; k < 4 && rc == WDIRAC_OK; ++k) rc = launch(k);
    if (rc == WDIRAC_OK && hipEventRecord(e0, st) != hipSuccess) rc = fail(WDIRAC_EHIP, "hipEventRecord");
    for (int k = 0; k < reps && rc == WDIRAC_OK; ++k) rc = launch(k);
    if (rc == WDIRAC_OK && hipEventRecord(e1, st) != hipSuccess) rc = fail(WDIRAC_EHIP, "hipEventRecord");
    if (rc == WDIRAC_OK && hipEventSynchronize(e1) != hipSuccess) rc = fail(WDIRAC_EHIP, "hipEventSynchronize");
    *ms = 0.0f;
    if (rc == WDIRAC_OK && hipEventElapsedTime(ms, e0, e1) != hipSuccess) rc = fail(WDIRAC_EHIP, "hipEventElapsedTime");
    *ms /= (float)reps;
  };
  // Pass 1: every candidate, 10 launches, then again over about 5 ms (at
  // most 100 launches), keeping the faster.  Pass 2: the best six again,
  // five interleaved rounds of at least 20 launches and about 25 ms each (so
  // that millisecond-scale kernels are timed over many launches), keeping
  // each one's fastest round; the spread of the pick's rounds is reported.
  std::vector<std::pair<float, int>> t1;
  {
    // untimed: about 50 ms of launches first, so that no candidate is timed
    // while the clocks are still ramping up
    float ms;
    time_cand(cands.front(), 4, &ms);
    if (rc == WDIRAC_OK) time_cand(cands.front(), std::min(1000, std::max(4, (int)(50.0f / std::max(ms, 1e-3f)))), &ms);
  }
  for (size_t i = 0; i < cands.size() && rc == WDIRAC_OK; ++i) {
    float ms, ms2 = 1e30f;
    time_cand(cands[i], 10, &ms);
    const int n2 = std::min(100, (int)(5.0f / std::max(ms, 1e-3f)));
    if (rc == WDIRAC_OK && n2 > 10) time_cand(cands[i], n2, &ms2);
    t1.push_back({std::min(ms, ms2), (int)i});
  }
  float best_ms = 1e30f, best_worst = 0.0f, second_ms = 0.0f;
  Cand pick = cands.front();
  if (rc == WDIRAC_OK) {
    std::sort(t1.begin(), t1.end());
    const size_t nfin = std::min<size_t>(6, t1.size());
    std::vector<float> t2(nfin, 1e30f), t2w(nfin, 0.0f);
    std::vector<int> reps(nfin);
    for (size_t j = 0; j < nfin; ++j)
      reps[j] = std::min(1000, std::max(20, (int)(25.0f / std::max(t1[j].first, 1e-3f))));
    for (int round = 0; round < 5 && rc == WDIRAC_OK; ++round)
      for (size_t j = 0; j < nfin && rc == WDIRAC_OK; ++j) {
        float ms;
        time_cand(cands[t1[j].second], reps[j], &ms);
        t2[j] = std::min(t2[j], ms);
        t2w[j] = std::max(t2w[j], ms);
      }
    size_t jb = 0;
    for (size_t j = 0; j < nfin; ++j)
      if (t2[j] < best_ms) {
        best_ms = t2[j];
        jb = j;
      }
    pick = cands[t1[jb].second];
    best_worst = t2w[jb];
    second_ms = 1e30f;
    for (size_t j = 0; j < nfin; ++j)
      if (j != jb) second_ms = std::min(second_ms, t2[j]);
    if (nfin < 2) second_ms = best_ms;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != WDIRAC_OK) {
    slot.valid = 0;
    return rc;
  }
  slot = wdirac_tuned{1, pick.variant, pick.nr, pick.remap, pick.tblock};
  if (best) {
    best->variant = pick.variant;
    best->nr = pick.nr;
    best->xcd_remap = pick.remap;
    best->tblock = pick.tblock;
    best->candidates = (int)cands.size();
    best->us = best_ms * 1e3;
    best->spread = best_ms > 0.0f ? (best_worst - best_ms) / best_ms : 0.0;
    best->runner_up_us = second_ms * 1e3;
  }
  return WDIRAC_OK;
}

int wdirac_pack_spinor(const wdirac_ctx *ctx, void *packed, const void *canon, int parity, int nrhs, int prec,
                       void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(packed, "packed"));
  WD_TRY(check_ptr(canon, "canon"));
  WD_TRY(check_parity(parity));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  return pack(ctx, packed, const_cast<void *>(canon), parity, nrhs, prec, 0, S(stream));
}

int wdirac_unpack_spinor(const wdirac_ctx *ctx, void *canon, const void *packed, int parity, int nrhs, int prec,
                         void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(packed, "packed"));
  WD_TRY(check_ptr(canon, "canon"));
  WD_TRY(check_parity(parity));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  return pack(ctx, const_cast<void *>(packed), canon, parity, nrhs, prec, 1, S(stream));
}

int wdirac_rep_links(const wdirac_ctx *ctx, void *UR, const void *U, int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(U, "U"));
  WD_TRY(check_prec(prec));
  const size_t el = (prec == WDIRAC_F64 ? 8 : 4) * (ctx->real ? 1 : 2);
  for (int l = 0; l < ctx->nlat; ++l) {
    const char *Ul = static_cast<const char *>(U) + (size_t)ctx->vpre[l] * 4 * ctx->N * ctx->N * 16;
    char *URl = static_cast<char *>(UR) + (size_t)8 * ctx->d * ctx->d * ctx->spre[l] * el;
    char *Fl = nullptr;
    if (wd::compact_links_ok(ctx->N, ctx->rep))
      Fl = static_cast<char *>(UR) + rep_links_bytes(ctx, prec) +
           (size_t)8 * ctx->N * ctx->N * ctx->spre[l] * (prec == WDIRAC_F64 ? 16 : 8);
    WD_HIP(wd::launch_rep_links(Ul, URl, Fl, ctx->g[l], ctx->N, ctx->rep, prec, S(stream)));
  }
  return WDIRAC_OK;
}

int wdirac_unpack_links(const wdirac_ctx *ctx, void *UR_canon, const void *UR, int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(UR_canon, "UR_canon"));
  WD_TRY(check_prec(prec));
  const size_t el = (prec == WDIRAC_F64 ? 8 : 4) * (ctx->real ? 1 : 2);
  const size_t cel = ctx->real ? 8 : 16;
  for (int l = 0; l < ctx->nlat; ++l) {
    char *Cl = static_cast<char *>(UR_canon) + (size_t)ctx->vpre[l] * 4 * ctx->d * ctx->d * cel;
    const char *URl = static_cast<const char *>(UR) + (size_t)8 * ctx->d * ctx->d * ctx->spre[l] * el;
    WD_HIP(wd::launch_unpack_links(Cl, URl, ctx->g[l], ctx->d, ctx->real, prec, S(stream)));
  }
  return WDIRAC_OK;
}

int wdirac_dslash_eo(const wdirac_ctx *ctx, void *out, const void *in, const void *UR, int out_parity, int dagger,
                     int nrhs, double alpha, const void *x_add, double beta, int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_parity(out_parity));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (dagger != 0 && dagger != 1) return fail(WDIRAC_EINVAL, "dagger must be 0 or 1");
  if (in == out) return fail(WDIRAC_EINVAL, "in and out must not alias");
  return hop(ctx, out, in, UR, out_parity, dagger, nrhs, alpha, x_add, beta, prec, nullptr, S(stream));
}

static int apply_M(const wdirac_ctx *ctx, void *out, const void *in, double m0, int inverse, int nrhs, int prec,
                   void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (inverse && 4.0 + m0 == 0.0) return fail(WDIRAC_EINVAL, "4 + m0 = 0 has no inverse");
  const double f = inverse ? 1.0 / (4.0 + m0) : 4.0 + m0;
  WD_HIP(wd::launch_lincomb(out, f, in, 0.0, nullptr, shape(ctx, nrhs), prec, S(stream)));
  return WDIRAC_OK;
}

int wdirac_apply_Mee(const wdirac_ctx *ctx, void *out, const void *in, double m0, int inverse, int nrhs, int prec,
                     void *stream) {
  return apply_M(ctx, out, in, m0, inverse, nrhs, prec, stream);
}

int wdirac_apply_Moo(const wdirac_ctx *ctx, void *out, const void *in, double m0, int inverse, int nrhs, int prec,
                     void *stream) {
  return apply_M(ctx, out, in, m0, inverse, nrhs, prec, stream);
}

int wdirac_apply_dhat(const wdirac_ctx *ctx, void *out, const void *in, const void *UR, double m0, int dagger,
                      int nrhs, int prec, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (dagger != 0 && dagger != 1) return fail(WDIRAC_EINVAL, "dagger must be 0 or 1");
  if (in == out) return fail(WDIRAC_EINVAL, "in and out must not alias");
  return dhat(ctx, out, in, UR, m0, dagger, nrhs, prec, workspace, nullptr, S(stream));
}

}  // extern "C"

// Scratch of wdirac_apply_dhat_noalloc: the odd half field between the two
// hops, in a device array of fixed size that every call on a GPU shares (each
// GPU holds its own copy from the first call until the process ends).  In
// host code `scratch` names a host-side stand-in; kernels receive the device
// address that hipGetSymbolAddress returns for the current device.
static constexpr size_t kNoallocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) char scratch[kNoallocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int scratch_address(void **out) {
  int dev = -1;
  WD_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(WDIRAC_EHIP, "device index out of range for the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    WD_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return fail(WDIRAC_EHIP, "hipGetSymbolAddress returned a null scratch address");
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return WDIRAC_OK;
}
}  // namespace

extern "C" {

size_t wdirac_noalloc_scratch_bytes(void) { return kNoallocScratchBytes; }

int wdirac_apply_dhat_noalloc(const wdirac_ctx *ctx, void *out, const void *in, const void *UR, double m0,
                              int dagger, int nrhs, int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (dagger != 0 && dagger != 1) return fail(WDIRAC_EINVAL, "dagger must be 0 or 1");
  if (in == out) return fail(WDIRAC_EINVAL, "in and out must not alias");
  const size_t need = half_bytes(ctx, nrhs, prec);
  if (need > kNoallocScratchBytes)
    return fail(WDIRAC_EINVAL, "apply_dhat_noalloc: the odd half field needs " + std::to_string(need) +
                                   " bytes, more than the " + std::to_string(kNoallocScratchBytes) +
                                   "-byte scratch; use wdirac_apply_dhat with a workspace");
  void *tmp = nullptr;
  WD_TRY(scratch_address(&tmp));
  // the first hop writes every element of tmp that the second reads: nothing
  // left by an earlier call needs clearing
  return dhat(ctx, out, in, UR, m0, dagger, nrhs, prec, tmp, nullptr, S(stream));
}

int wdirac_eo_source(const wdirac_ctx *ctx, void *b_e, const void *eta_e, const void *eta_o, const void *UR,
                     double m0, int nrhs, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(b_e, "b_e"));
  WD_TRY(check_ptr(eta_e, "eta_e"));
  WD_TRY(check_ptr(eta_o, "eta_o"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_nrhs(ctx, nrhs));
  if (b_e == eta_o) return fail(WDIRAC_EINVAL, "b_e must not alias eta_o");
  return hop(ctx, b_e, eta_o, UR, 0, 0, nrhs, 4.0 + m0, eta_e, -1.0, WDIRAC_F64, nullptr, S(stream));
}

int wdirac_eo_reconstruct(const wdirac_ctx *ctx, void *psi_o, const void *psi_e, const void *eta_o, const void *UR,
                          double m0, int nrhs, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(psi_o, "psi_o"));
  WD_TRY(check_ptr(psi_e, "psi_e"));
  WD_TRY(check_ptr(eta_o, "eta_o"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_nrhs(ctx, nrhs));
  if (4.0 + m0 == 0.0) return fail(WDIRAC_EINVAL, "4 + m0 = 0 has no inverse");
  if (psi_o == psi_e) return fail(WDIRAC_EINVAL, "psi_o must not alias psi_e");
  const double f = 1.0 / (4.0 + m0);
  return hop(ctx, psi_o, psi_e, UR, 1, 0, nrhs, f, eta_o, -f, WDIRAC_F64, nullptr, S(stream));
}

int wdirac_norm2(const wdirac_ctx *ctx, double *out, const void *v, int nrhs, int prec, void *workspace,
                 void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(v, "v"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  Carver cv{static_cast<char *>(workspace)};
  double *part = static_cast<double *>(cv.take(partial_doubles(ctx, nrhs) * sizeof(double)));
  double *dout = static_cast<double *>(cv.take(2 * wd::MAXSYS * sizeof(double)));
  const wd::FieldShape f = shape(ctx, nrhs);
  const int nb = wd::blas_nblocks(f);
  WD_HIP(wd::launch_norm2_partial(part, v, f, prec, S(stream)));
  WD_HIP(wd::launch_finalize_sum(dout, part, nb, wd::uniform_counts(nb), f.nsys, f.nsys, S(stream)));
  WD_HIP(hipMemcpyAsync(out, dout, f.nsys * sizeof(double), hipMemcpyDeviceToHost, S(stream)));
  WD_HIP(hipStreamSynchronize(S(stream)));
  return WDIRAC_OK;
}

int wdirac_dot(const wdirac_ctx *ctx, double *out, const void *a, const void *b, int nrhs, int prec, void *workspace,
               void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(a, "a"));
  WD_TRY(check_ptr(b, "b"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  Carver cv{static_cast<char *>(workspace)};
  double *part = static_cast<double *>(cv.take(partial_doubles(ctx, nrhs) * sizeof(double)));
  double *dout = static_cast<double *>(cv.take(2 * wd::MAXSYS * sizeof(double)));
  const wd::FieldShape f = shape(ctx, nrhs);
  const int nb = wd::blas_nblocks(f), ns = f.nsys;
  WD_HIP(wd::launch_dot_partial(part, a, b, f, prec, S(stream)));
  WD_HIP(wd::launch_finalize_sum(dout, part, nb, wd::uniform_counts(nb), 2 * ns, ns, S(stream)));
  std::vector<double> tmp(2 * ns);
  WD_HIP(hipMemcpyAsync(tmp.data(), dout, 2 * ns * sizeof(double), hipMemcpyDeviceToHost, S(stream)));
  WD_HIP(hipStreamSynchronize(S(stream)));
  for (int k = 0; k < ns; ++k) {
    out[2 * k] = tmp[k];
    out[2 * k + 1] = tmp[ns + k];
  }
  return WDIRAC_OK;
}

// ------------------------------------------------------------------- CG
// Per right-hand side, the Hestenes-Stiefel recurrence on A = D-hat^+ D-hat:
//   q = A p (u = D-hat p gives <p, A p> = ||u||^2, then q = D-hat^+ u),
//   alpha = rho / <p,Ap>;  x += alpha p;  r -= alpha q;  rho' = ||r||^2;
//   beta = rho'/rho;  p = r + beta p.
// All scalars stay on the device; kernels of right-hand sides that are done
// return at once, so the host only reads the scalars every few iterations.
// When the recursive residual reaches the target, r is recomputed as b - A x
// in FP64 (the "true" residual); if it is above target the recurrence resumes
// from it with p kept (residual replacement).  Mixed mode runs the
// recurrence in FP32 (hops, vectors; sums in FP64) on the correction
// equation and replaces the residual in FP64 whenever ||r|| drops below
// delta times its largest value since the previous replacement (reliable
// updates), accumulating the FP32 correction into the FP64 solution.
static int cg_impl(const wdirac_ctx *ctx, void *x, const void *b, const void *UR64, const void *UR32,
                   const void *clov64, const void *clov32, double m0, double tol, int maxit, int nrhs, int mode,
                   void *workspace, wdirac_cg_stats *stats, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(x, "x"));
  WD_TRY(check_ptr(b, "b"));
  WD_TRY(check_ptr(UR64, "UR64"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_ptr(stats, "stats"));
  WD_TRY(check_nrhs(ctx, nrhs));
  if (mode != WDIRAC_CG_F64 && mode != WDIRAC_CG_MIXED) return fail(WDIRAC_EINVAL, "unknown CG mode");
  if (mode == WDIRAC_CG_MIXED) WD_TRY(check_ptr(UR32, "UR32"));
  if (!(tol > 0.0) || maxit < 0) return fail(WDIRAC_EINVAL, "tol must be > 0 and maxit >= 0");
  if (x == b) return fail(WDIRAC_EINVAL, "x and b must not alias");
  hipStream_t st = S(stream);
  // the solve starts once the caller's queued work is done: the reported
  // time is that of the solve alone
  WD_HIP(hipStreamSynchronize(st));
  const auto t0 = std::chrono::steady_clock::now();
  if (ctx->cg_graph) {
    // the iterations between host checks are captured once and replayed as
    // a graph; capture needs a stream of the library's own (the caller's may
    // be the null stream), ordered after the caller's work (drained above)
    if (!ctx->own && hipStreamCreateWithFlags(&ctx->own, hipStreamNonBlocking) != hipSuccess) ctx->own = nullptr;
    if (ctx->own) st = ctx->own;
  }
  const bool mixed = mode == WDIRAC_CG_MIXED;
  CgWork w = carve_cg(ctx, nrhs, mode, workspace);
  const wd::FieldShape f = shape(ctx, nrhs);
  const int nbb = wd::blas_nblocks(f), ns = f.nsys;
  std::vector<wd::CgScalars> hs(ns);
  std::vector<int> rel(ns, 0);
  int hop_count = 0, updates = 0;

  // b2, stop2
  wd::Counts rcnt = wd::uniform_counts(nbb);   // partial sums of |r|^2 in w.P2: per system, and their row length
  int rprow = nbb;
  WD_HIP(wd::launch_norm2_partial(w.P2, b, f, WDIRAC_F64, st));
  WD_HIP(wd::launch_cg_restart(w.sc, w.P2, rprow, rcnt, ns, tol, 1, st));
  // r = b - A x (FP64)
  auto true_residual = [&]() -> int {
    CgHop cr;
    cr.r = w.r;
    cr.rin = b;
    WD_TRY(dhat(ctx, w.u, x, UR64, m0, 0, nrhs, WDIRAC_F64, w.t, nullptr, st, nullptr, nullptr, clov64));
    WD_TRY(dhat(ctx, w.q, w.u, UR64, m0, 1, nrhs, WDIRAC_F64, w.v, w.P2, st, &rcnt, &rprow, clov64, nullptr, &cr));
    hop_count += 4;
    return WDIRAC_OK;
  };
  WD_TRY(true_residual());
  WD_HIP(wd::launch_cg_restart(w.sc, w.P2, rprow, rcnt, ns, tol, 0, st));
  void *r = w.r, *p = w.p, *q = w.q, *t = w.t, *u = w.u, *v = w.v, *xi = x;
  const void *UR = UR64, *clov = clov64;
  int prec = WDIRAC_F64;
  if (mixed) {
    WD_HIP(wd::launch_convert(w.r32, WDIRAC_F32, w.r, WDIRAC_F64, f, st));
    WD_HIP(wd::launch_lincomb(w.x32, 0.0, w.r32, 0.0, nullptr, f, WDIRAC_F32, st));
    r = w.r32; p = w.p32; q = w.q32; t = w.t32; u = w.u32; v = w.v32; xi = w.x32;
    UR = UR32;
    clov = clov32;
    prec = WDIRAC_F32;
  }
  WD_HIP(wd::launch_lincomb(p, 1.0, r, 0.0, nullptr, f, prec, st));
  const double delta = mixed ? ctx->mixed_delta : 0.0;
  int rc = WDIRAC_OK;
  int launched = 0;   // iterations launched since start
  // lattices that fit one workgroup iterate inside one kernel until they stop
  // (mixed mode: from check to check, where replacements are decided)
  const bool tiny = ctx->nlat == 1 && !clov64 && wd::cg_tiny_ok(ctx->g[0], ctx->d, ctx->real);
  const int check = check_every(ctx, tiny && !mixed);
  int seen_iters = 0;   // hops counted so far (tiny)
  bool use_graph = ctx->cg_graph && st == ctx->own && !tiny;
  hipGraphExec_t exec = nullptr;
  for (;;) {
    WD_HIP(hipMemcpyAsync(hs.data(), w.sc, ns * sizeof(wd::CgScalars), hipMemcpyDeviceToHost, st));
    WD_HIP(hipStreamSynchronize(st));
    // a residual replacement runs once every system that is still iterating
    // has asked for one (mixed mode) or has stopped (converged recursion,
    // breakdown)
    bool any_active = false, any_update = false, all_ready = true;
    for (int k = 0; k < ns; ++k) {
      any_active |= hs[k].active != 0;
      any_update |= hs[k].need_update != 0;
      all_ready &= hs[k].active == 0 || hs[k].need_update != 0;
    }
    int max_iters = 0;
    for (int k = 0; k < ns; ++k) max_iters = std::max(max_iters, hs[k].iters);
    if (tiny) {
      hop_count += 4 * (max_iters - seen_iters);
      seen_iters = max_iters;
    }
    if (any_update && all_ready) {
      // residual replacement in FP64 (verifies convergence of the recursion)
      if (mixed) WD_HIP(wd::launch_accum_x(x, w.x32, f, st));
      WD_TRY(true_residual());
      WD_HIP(wd::launch_cg_restart(w.sc, w.P2, rprow, rcnt, ns, tol, 0, st));
      if (mixed) WD_HIP(wd::launch_convert(w.r32, WDIRAC_F32, w.r, WDIRAC_F64, f, st));
      ++updates;
      for (int k = 0; k < ns; ++k)
        if (hs[k].need_update) ++rel[k];
      continue;
    }
    if (!any_active) break;
    if (max_iters >= maxit) {
      rc = WDIRAC_ENOCONV;
      break;
    }
    const int nit = std::min(check, std::max(1, maxit - max_iters));
    if (tiny) {
      const double m4 = (4.0 + m0) * (4.0 + m0);
      WD_HIP(wd::launch_cg_tiny(xi, p, r, UR, ctx->g[0], ctx->d, ctx->real, w.sc, m4, delta, nit, nrhs, prec, st));
      continue;
    }
    auto launch_iters = [&](int n) -> int {
      for (int it = 0; it < n; ++it) {
        wd::Counts cnt{};
        int prow = 0;
        // u = D-hat p with ||u||^2; then A p = D-hat^+ u: alpha beside the
        // first of its hops, r -= alpha A p in the second (A p itself is not
        // stored; q holds D_ee u of the clover form)
        WD_TRY(dhat(ctx, u, p, UR, m0, 0, nrhs, prec, t, w.P1, st, &cnt, &prow, clov));
        CgHop ca, cr;
        ca.sc = cr.sc = w.sc;
        ca.lead = ns;
        ca.lp = w.P1;
        ca.lprow = prow;
        ca.lcnt = cnt;
        cr.r = r;
        cr.rin = r;
        WD_TRY(dhat(ctx, q, u, UR, m0, 1, nrhs, prec, v, w.P2, st, &cnt, &prow, clov, &ca, &cr));
        WD_HIP(wd::launch_cg_update_xp(xi, p, r, w.sc, w.P2, prow, cnt, delta, f, prec, st));
      }
      return WDIRAC_OK;
    };
    if (use_graph && nit == check && !exec) {
      hipGraph_t graph = nullptr;
      if (hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) == hipSuccess) {
        const int crc = launch_iters(nit);
        const hipError_t ce = hipStreamEndCapture(st, &graph);
        if (crc != WDIRAC_OK || ce != hipSuccess || !graph ||
            hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess)
          exec = nullptr;
        if (graph) (void)hipGraphDestroy(graph);
      }
      if (!exec) {
        use_graph = false;   // capture unavailable: launch directly from now on
        g_err.clear();
      }
    }
    if (use_graph && nit == check && exec) WD_HIP(hipGraphLaunch(exec, st));
    else WD_TRY(launch_iters(nit));
    hop_count += 4 * nit;
    launched += nit;
  }
  if (exec) (void)hipGraphExecDestroy(exec);
  if (mixed) WD_HIP(wd::launch_accum_x(x, w.x32, f, st));
  // final FP64 true residual of the returned x
  WD_TRY(true_residual());
  WD_HIP(wd::launch_finalize_sum(w.P1, w.P2, rprow, rcnt, ns, ns, st));
  std::vector<double> res2(ns);
  WD_HIP(hipMemcpyAsync(res2.data(), w.P1, ns * sizeof(double), hipMemcpyDeviceToHost, st));
  WD_HIP(hipMemcpyAsync(hs.data(), w.sc, ns * sizeof(wd::CgScalars), hipMemcpyDeviceToHost, st));
  WD_HIP(hipStreamSynchronize(st));
  // b = 0: the solution is x = 0 whatever the initial guess
  for (int k = 0; k < ns; ++k)
    if (!(hs[k].b2 > 0.0)) {
      const size_t bytes = (size_t)f.ncomp * f.stride[k] * 16;
      WD_HIP(hipMemsetAsync(static_cast<char *>(x) + (size_t)f.off[k] * 16, 0, bytes, st));
      res2[k] = 0.0;
    }
  WD_HIP(hipStreamSynchronize(st));
  const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  int worst = WDIRAC_OK;
  for (int k = 0; k < ns; ++k) {
    wdirac_cg_stats &s = stats[k];
    s.iters = hs[k].iters;
    s.reliable_updates = rel[k];
    s.hops = hop_count;
    s.true_rel_resid = hs[k].b2 > 0.0 ? std::sqrt(res2[k] / hs[k].b2) : 0.0;
    s.seconds = secs;
    int stk = hs[k].status;
    if (stk == WDIRAC_OK && hs[k].b2 > 0.0 && !(s.true_rel_resid <= tol)) stk = WDIRAC_ENOCONV;
    s.status = stk;
    if (stk == WDIRAC_EBREAKDOWN) worst = WDIRAC_EBREAKDOWN;
    else if (stk == WDIRAC_ENOCONV && worst == WDIRAC_OK) worst = WDIRAC_ENOCONV;
  }
  (void)launched;
  (void)updates;
  if (rc == WDIRAC_ENOCONV && worst == WDIRAC_OK) worst = WDIRAC_ENOCONV;
  if (worst == WDIRAC_ENOCONV) fail(worst, "CG did not reach the tolerance within maxit");
  if (worst == WDIRAC_EBREAKDOWN) fail(worst, "CG breakdown (non-finite value or <p,Ap> <= 0)");
  return worst;
}

int wdirac_cg_eo(const wdirac_ctx *ctx, void *x, const void *b, const void *UR64, const void *UR32, double m0,
                 double tol, int maxit, int nrhs, int mode, void *workspace, wdirac_cg_stats *stats, void *stream) {
  return cg_impl(ctx, x, b, UR64, UR32, nullptr, nullptr, m0, tol, maxit, nrhs, mode, workspace, stats, stream);
}

// ------------------------------------------------------------------ clover
int wdirac_clover_field(const wdirac_ctx *ctx, void *clov, const void *U, double m0, double csw, int exponential,
                        int prec, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(clov, "clov"));
  WD_TRY(check_ptr(U, "U"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_prec(prec));
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  if (!std::isfinite(m0) || !std::isfinite(csw) || 4.0 + m0 == 0.0)
    return fail(WDIRAC_EINVAL, "m0 and csw must be finite and 4 + m0 != 0");
  if (exponential != 0 && exponential != 1) return fail(WDIRAC_EINVAL, "exponential must be 0 or 1");
  const size_t el = prec == WDIRAC_F64 ? 8 : 4;
  for (int l = 0; l < ctx->nlat; ++l) {
    const char *Ul = static_cast<const char *>(U) + (size_t)ctx->vpre[l] * 4 * ctx->N * ctx->N * 16;
    char *cl = static_cast<char *>(clov) + (size_t)4 * ctx->d * (2 * ctx->d + 1) * ctx->spre[l] * 2 * el;
    int mx = 0;
    for (int k = 0; k < ctx->nlat; ++k) mx = std::max(mx, ctx->g[k].Vh);
    double *Fw = static_cast<double *>(workspace);
    double *Us = reinterpret_cast<double *>(static_cast<char *>(workspace) +
                                            align256((size_t)6 * ctx->d * ctx->d * 2 * mx * 16));
    WD_HIP(wd::launch_clover_field(cl, Ul, Fw, Us, ctx->g[l], ctx->N, ctx->rep, ctx->d, m0, csw, exponential, prec,
                                   S(stream)));
  }
  return WDIRAC_OK;
}

int wdirac_apply_clover(const wdirac_ctx *ctx, void *out, const void *in, const void *clov, int parity, int nrhs,
                        int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(clov, "clov"));
  WD_TRY(check_parity(parity));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  return clover_apply(ctx, out, in, clov, parity, nrhs, prec, S(stream));
}

int wdirac_apply_dhat_clover(const wdirac_ctx *ctx, void *out, const void *in, const void *UR, const void *clov,
                             int dagger, int nrhs, int prec, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(clov, "clov"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (dagger != 0 && dagger != 1) return fail(WDIRAC_EINVAL, "dagger must be 0 or 1");
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  if (out == in) return fail(WDIRAC_EINVAL, "out must not alias in");
  return dhat(ctx, out, in, UR, 0.0, dagger, nrhs, prec, workspace, nullptr, S(stream), nullptr, nullptr, clov);
}

int wdirac_cg_eo_clover(const wdirac_ctx *ctx, void *x, const void *b, const void *UR64, const void *UR32,
                        const void *clov64, const void *clov32, double tol, int maxit, int nrhs, int mode,
                        void *workspace, wdirac_cg_stats *stats, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(clov64, "clov64"));
  if (mode == WDIRAC_CG_MIXED) WD_TRY(check_ptr(clov32, "clov32"));
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  return cg_impl(ctx, x, b, UR64, UR32, clov64, clov32, 0.0, tol, maxit, nrhs, mode, workspace, stats, stream);
}

// ------------------------------------------------------------ multi-shift CG
int wdirac_cg_mshift_eo(const wdirac_ctx *ctx, void *x, const void *b, const void *UR64, double m0,
                        const double *shifts, int nshift, double tol, int maxit, void *workspace,
                        wdirac_cg_stats *stats, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(x, "x"));
  WD_TRY(check_ptr(b, "b"));
  WD_TRY(check_ptr(UR64, "UR64"));
  WD_TRY(check_ptr(shifts, "shifts"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_ptr(stats, "stats"));
  if (ctx->nlat != 1) return fail(WDIRAC_EUNSUPPORTED, "multi-shift CG runs on a single lattice");
  if (nshift < 1 || nshift > wd::MAXSHIFT) return fail(WDIRAC_EINVAL, "nshift must be in [1, 32]");
  if (!(tol > 0.0) || maxit < 0) return fail(WDIRAC_EINVAL, "tol must be > 0 and maxit >= 0");
  int base = 0;
  for (int k = 0; k < nshift; ++k) {
    if (!(shifts[k] >= 0.0) || !std::isfinite(shifts[k])) return fail(WDIRAC_EINVAL, "shifts must be finite and >= 0");
    if (shifts[k] < shifts[base]) base = k;
  }
  const size_t hb = half_bytes(ctx, 1, WDIRAC_F64);
  {
    const char *xs = static_cast<const char *>(x), *bs = static_cast<const char *>(b);
    if (bs + hb > xs && bs < xs + (size_t)nshift * hb) return fail(WDIRAC_EINVAL, "x and b must not overlap");
  }
  const hipStream_t st = S(stream);
  WD_HIP(hipStreamSynchronize(st));   // time the solve alone
  const auto t0 = std::chrono::steady_clock::now();
  MsWork w = carve_ms(ctx, nshift, workspace);
  const wd::FieldShape f = shape(ctx, 1);
  const int nbb = wd::blas_nblocks(f);
  const double sigma0 = shifts[base];
  const long long fstride = (long long)(hb / 16);
  wd::ShiftList dl{};
  for (int k = 0; k < nshift; ++k) dl.v[k] = shifts[k] - sigma0;
  auto field = [&](void *base_ptr, int k) { return static_cast<void *>(static_cast<char *>(base_ptr) + (size_t)k * hb); };
  // x_k = 0 (padding included), p_k = b, r = b
  WD_HIP(hipMemsetAsync(x, 0, (size_t)nshift * hb, st));
  WD_HIP(wd::launch_lincomb(field(w.r, w.ring - 1), 1.0, b, 0.0, nullptr, f, WDIRAC_F64, st));
  for (int k = 0; k < nshift; ++k) WD_HIP(wd::launch_lincomb(field(w.p, k), 1.0, b, 0.0, nullptr, f, WDIRAC_F64, st));
  WD_HIP(wd::launch_norm2_partial(w.P2, b, f, WDIRAC_F64, st));
  // the recursion stops at half the tolerance, leaving room for the drift of
  // the recursive residuals from the true ones checked below
  WD_HIP(wd::launch_ms_init(w.sc, w.P2, nbb, dl, nshift, base, sigma0, 0.5 * tol, st));
  int hop_count = 0, rc = WDIRAC_OK;
  wd::MsScalars hs{};
  void *pb = field(w.p, base), *xb = field(x, base);
  // |p|^2 of the next step length (sigma0 > 0): at first that of b
  const double *pp = w.P2;
  int npp = nbb, slot = 0;
  const auto flush = [&]() -> int {   // the other shifts' updates of the iterations in the ring
    if (slot && nshift > 1)
      WD_HIP(wd::launch_ms_update_xp(x, w.p, w.r, w.sc, fstride, f, slot, st));
    slot = 0;
    return WDIRAC_OK;
  };
  for (;;) {
    WD_HIP(hipMemcpyAsync(&hs, w.sc, sizeof(hs), hipMemcpyDeviceToHost, st));
    WD_HIP(hipStreamSynchronize(st));
    if (!hs.cg.active) break;
    if (hs.cg.iters >= maxit) {
      rc = WDIRAC_ENOCONV;
      break;
    }
    const int nit = std::min(check_every(ctx, false), std::max(1, maxit - hs.cg.iters));
    for (int it = 0; it < nit; ++it) {
      wd::Counts cnt{};
      int prow = 0;
      WD_TRY(dhat(ctx, w.u, pb, UR64, m0, 0, 1, WDIRAC_F64, w.t, w.P1, st, &cnt, &prow));
      CgHop ca, cr;
      ca.lead = 1;
      ca.ms = w.sc;
      ca.lp = w.P1;
      ca.lprow = prow;
      ca.lcnt = cnt;
      cr.sc = &w.sc->cg;
      cr.rin = field(w.r, (slot + w.ring - 1) % w.ring);
      cr.r = field(w.r, slot % w.ring);
      if (sigma0 != 0.0) {
        ca.lp2 = pp;
        ca.lcnt2 = npp;
        cr.ps = pb;
        cr.sigma = sigma0;
      }
      // (w.u is only the hop's nominal output: r is stored in its place)
      WD_TRY(dhat(ctx, w.u, w.u, UR64, m0, 1, 1, WDIRAC_F64, w.t, w.P2, st, &cnt, &prow, nullptr, &ca, &cr));
      WD_HIP(wd::launch_ms_update_base(xb, pb, cr.r, w.sc, w.P2, cnt.n[0], slot, sigma0 != 0.0 ? w.P3 : nullptr, f,
                                       st));
      pp = w.P3;
      npp = wd::ms_base_blocks(f);
      if (++slot == w.ring) WD_TRY(flush());
      hop_count += 4;
    }
  }
  WD_TRY(flush());
  // true residuals ||b - (A + sigma_k) x_k||
  std::vector<double> res2(nshift);
  for (int k = 0; k < nshift; ++k) {
    wd::Counts cnt{};
    int prow = 0;
    CgHop cr;
    cr.r = w.r;
    cr.rin = b;
    cr.ps = field(x, k);
    cr.sigma = shifts[k];
    WD_TRY(dhat(ctx, w.u, field(x, k), UR64, m0, 0, 1, WDIRAC_F64, w.t, nullptr, st));
    WD_TRY(dhat(ctx, w.u, w.u, UR64, m0, 1, 1, WDIRAC_F64, w.t, w.P2, st, &cnt, &prow, nullptr, nullptr, &cr));
    WD_HIP(wd::launch_finalize_sum(w.P1, w.P2, prow, cnt, 1, 1, st));
    WD_HIP(hipMemcpyAsync(&res2[k], w.P1, sizeof(double), hipMemcpyDeviceToHost, st));
    hop_count += 4;
  }
  WD_HIP(hipMemcpyAsync(&hs, w.sc, sizeof(hs), hipMemcpyDeviceToHost, st));
  WD_HIP(hipStreamSynchronize(st));
  const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  int worst = WDIRAC_OK;
  for (int k = 0; k < nshift; ++k) {
    wdirac_cg_stats &sk = stats[k];
    sk.iters = hs.siters[k];
    sk.reliable_updates = 0;
    sk.hops = hop_count;
    sk.true_rel_resid = hs.cg.b2 > 0.0 ? std::sqrt(res2[k] / hs.cg.b2) : 0.0;
    sk.seconds = secs;
    int stk = hs.cg.status;
    if (stk == WDIRAC_OK && hs.cg.b2 > 0.0 && (hs.sact[k] || !(sk.true_rel_resid <= tol))) stk = WDIRAC_ENOCONV;
    sk.status = stk;
    if (stk == WDIRAC_EBREAKDOWN) worst = WDIRAC_EBREAKDOWN;
    else if (stk == WDIRAC_ENOCONV && worst == WDIRAC_OK) worst = WDIRAC_ENOCONV;
  }
  if (rc == WDIRAC_ENOCONV && worst == WDIRAC_OK) worst = WDIRAC_ENOCONV;
  if (worst == WDIRAC_ENOCONV) fail(worst, "multi-shift CG: some shift did not reach the tolerance");
  if (worst == WDIRAC_EBREAKDOWN) fail(worst, "multi-shift CG breakdown (non-finite value or <p,Ap> <= 0)");
  return worst;
}

int wdirac_axpby(const wdirac_ctx *ctx, void *out, double a, const void *x, double b, const void *y, int nrhs,
                 int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(x, "x"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  WD_HIP(wd::launch_lincomb(out, a, x, b, y, shape(ctx, nrhs), prec, S(stream)));
  return WDIRAC_OK;
}

// ------------------------------------------------------------- HMC pieces
static size_t links_offset(const wdirac_ctx *c, int l) { return (size_t)c->vpre[l] * 4 * c->N * c->N * 16; }

int wdirac_gauge_force(const wdirac_ctx *ctx, void *F, const void *U, double beta, double scale, int accumulate,
                       void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(F, "F"));
  WD_TRY(check_ptr(U, "U"));
  if (accumulate != 0 && accumulate != 1) return fail(WDIRAC_EINVAL, "accumulate must be 0 or 1");
  if (F == U) return fail(WDIRAC_EINVAL, "F must not alias U");
  for (int l = 0; l < ctx->nlat; ++l)
    WD_HIP(wd::launch_gauge_force(static_cast<const char *>(U) + links_offset(ctx, l),
                                  static_cast<char *>(F) + links_offset(ctx, l), ctx->g[l], ctx->N, beta, scale,
                                  accumulate, S(stream)));
  return WDIRAC_OK;
}

// Sum of the block partials (FP64, compensated) to the host.
static int reduce_to_host(double *out, const double *partial, int nblk, double *dtmp, hipStream_t st) {
  WD_HIP(wd::launch_finalize_sum(dtmp, partial, nblk, wd::uniform_counts(nblk), 1, 1, st));
  WD_HIP(hipMemcpyAsync(out, dtmp, sizeof(double), hipMemcpyDeviceToHost, st));
  WD_HIP(hipStreamSynchronize(st));
  return WDIRAC_OK;
}

int wdirac_gauge_action(const wdirac_ctx *ctx, double *S_out, const void *U, double beta, void *workspace,
                        void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(S_out, "S"));
  WD_TRY(check_ptr(U, "U"));
  WD_TRY(check_ptr(workspace, "workspace"));
  Carver cv{static_cast<char *>(workspace)};
  int mx = 0;
  for (int l = 0; l < ctx->nlat; ++l) mx = std::max(mx, wd::kinetic_blocks(ctx->g[l]));
  double *part = static_cast<double *>(cv.take((size_t)mx * sizeof(double)));
  double *dtmp = static_cast<double *>(cv.take(sizeof(double)));
  for (int l = 0; l < ctx->nlat; ++l) {
    const int nb = wd::plaquette_blocks(ctx->g[l]);
    WD_HIP(wd::launch_plaquette_partial(static_cast<const char *>(U) + links_offset(ctx, l), part, ctx->g[l],
                                        ctx->N, S(stream)));
    double plaq = 0.0;
    WD_TRY(reduce_to_host(&plaq, part, nb, dtmp, S(stream)));
    S_out[l] = beta * (6.0 * 2.0 * ctx->g[l].Vh - plaq);
  }
  return WDIRAC_OK;
}

int wdirac_link_update(const wdirac_ctx *ctx, void *U, const void *pi, double eps, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(U, "U"));
  WD_TRY(check_ptr(pi, "pi"));
  if (U == pi) return fail(WDIRAC_EINVAL, "pi must not alias U");
  if (!std::isfinite(eps)) return fail(WDIRAC_EINVAL, "eps must be finite");
  for (int l = 0; l < ctx->nlat; ++l)
    WD_HIP(wd::launch_link_update(static_cast<char *>(U) + links_offset(ctx, l),
                                  static_cast<const char *>(pi) + links_offset(ctx, l), ctx->g[l], ctx->N, eps,
                                  S(stream)));
  return WDIRAC_OK;
}

int wdirac_kinetic(const wdirac_ctx *ctx, double *K, const void *pi, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(K, "K"));
  WD_TRY(check_ptr(pi, "pi"));
  WD_TRY(check_ptr(workspace, "workspace"));
  Carver cv{static_cast<char *>(workspace)};
  int mx = 0;
  for (int l = 0; l < ctx->nlat; ++l) mx = std::max(mx, wd::kinetic_blocks(ctx->g[l]));
  double *part = static_cast<double *>(cv.take((size_t)mx * sizeof(double)));
  double *dtmp = static_cast<double *>(cv.take(sizeof(double)));
  for (int l = 0; l < ctx->nlat; ++l) {
    WD_HIP(wd::launch_kinetic_partial(static_cast<const char *>(pi) + links_offset(ctx, l), part, ctx->g[l], ctx->N,
                                      S(stream)));
    WD_TRY(reduce_to_host(&K[l], part, wd::kinetic_blocks(ctx->g[l]), dtmp, S(stream)));
  }
  return WDIRAC_OK;
}

int wdirac_algebra_from_components(const wdirac_ctx *ctx, void *pi, const double *w, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(pi, "pi"));
  WD_TRY(check_ptr(w, "w"));
  const int na = ctx->N * ctx->N - 1;
  for (int l = 0; l < ctx->nlat; ++l)
    WD_HIP(wd::launch_algebra(static_cast<char *>(pi) + links_offset(ctx, l), w + (size_t)ctx->vpre[l] * 4 * na,
                              ctx->g[l], ctx->N, S(stream)));
  return WDIRAC_OK;
}

// ---------------------------------------------- twisted mass, Hasenbusch
int wdirac_gamma5(const wdirac_ctx *ctx, void *out, const void *in, int nrhs, int prec, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  WD_HIP(wd::launch_gamma5_axpy(out, in, 0.0, nullptr, shape(ctx, nrhs), prec, S(stream)));
  return WDIRAC_OK;
}

int wdirac_apply_W(const wdirac_ctx *ctx, void *out, const void *in, const void *UR, double m0, double mu, int sign,
                   int nrhs, int prec, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(out, "out"));
  WD_TRY(check_ptr(in, "in"));
  WD_TRY(check_ptr(UR, "UR"));
  WD_TRY(check_ptr(workspace, "workspace"));
  WD_TRY(check_nrhs(ctx, nrhs));
  WD_TRY(check_prec(prec));
  if (sign != 1 && sign != -1) return fail(WDIRAC_EINVAL, "sign must be +1 or -1");
  if (!std::isfinite(mu)) return fail(WDIRAC_EINVAL, "mu must be finite");
  if (out == in) return fail(WDIRAC_EINVAL, "out must not alias in");
  const hipStream_t st = S(stream);
  WD_TRY(dhat(ctx, out, in, UR, m0, 0, nrhs, prec, workspace, nullptr, st));
  WD_HIP(wd::launch_gamma5_axpy(out, out, sign * mu, in, shape(ctx, nrhs), prec, st));
  return WDIRAC_OK;
}

int wdirac_force_bilinear_eo(const wdirac_ctx *ctx, void *P, const void *X_e, const void *X_o, const void *Y_e,
                             const void *Y_o, const void *UR64, const void *U, double scale, int accumulate,
                             void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(P, "out"));
  WD_TRY(check_ptr(X_e, "X_e"));
  WD_TRY(check_ptr(X_o, "X_o"));
  WD_TRY(check_ptr(Y_e, "Y_e"));
  WD_TRY(check_ptr(Y_o, "Y_o"));
  WD_TRY(check_ptr(UR64, "UR64"));
  if (accumulate != 0 && accumulate != 1) return fail(WDIRAC_EINVAL, "accumulate must be 0 or 1");
  const hipStream_t st = S(stream);
  const size_t el = ctx->real ? 8 : 16;
  for (int l = 0; l < ctx->nlat; ++l) {
    const size_t so = (size_t)4 * ctx->d * ctx->spre[l] * 16;
    const size_t po = (size_t)ctx->vpre[l] * 4 * ctx->N * ctx->N * 16;
    auto at = [so](const void *p) { return static_cast<const void *>(static_cast<const char *>(p) + so); };
    WD_HIP(wd::launch_force_links(static_cast<char *>(P) + po, at(X_e), at(X_o), at(Y_e), at(Y_o),
                                  static_cast<const char *>(UR64) + (size_t)8 * ctx->d * ctx->d * ctx->spre[l] * el,
                                  U ? static_cast<const char *>(U) + po : nullptr, ctx->g[l], ctx->N, ctx->rep, scale,
                                  accumulate, st));
  }
  WD_HIP(hipStreamSynchronize(st));
  return WDIRAC_OK;
}

int wdirac_force_eo(const wdirac_ctx *ctx, void *P, const void *x_e, const void *UR64, const void *U, double m0,
                    double scale, int accumulate, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(P, "out"));
  WD_TRY(check_ptr(x_e, "x_e"));
  WD_TRY(check_ptr(UR64, "UR64"));
  WD_TRY(check_ptr(workspace, "workspace"));
  const hipStream_t st = S(stream);
  Carver cv{static_cast<char *>(workspace)};
  const size_t h = half_bytes(ctx, 1, WDIRAC_F64);
  void *z_o = cv.take(h), *y_e = cv.take(h), *w_o = cv.take(h);
  // z_o = D_oe x;  y_e = (4+m)^2 x - D_eo z_o = D-hat x;  w_o = D_eo^+ y_e
  WD_TRY(hop(ctx, z_o, x_e, UR64, 1, 0, 1, 0.0, nullptr, 1.0, WDIRAC_F64, nullptr, st));
  WD_TRY(hop(ctx, y_e, z_o, UR64, 0, 0, 1, (4.0 + m0) * (4.0 + m0), x_e, -1.0, WDIRAC_F64, nullptr, st));
  WD_TRY(hop(ctx, w_o, y_e, UR64, 1, 1, 1, 0.0, nullptr, 1.0, WDIRAC_F64, nullptr, st));
  const size_t el = ctx->real ? 8 : 16;
  for (int l = 0; l < ctx->nlat; ++l) {
    const size_t so = (size_t)4 * ctx->d * ctx->spre[l] * 16;   // this lattice in the FP64 half fields
    const size_t po = (size_t)ctx->vpre[l] * 4 * ctx->N * ctx->N * 16;
    auto at = [so](const void *p) { return static_cast<const void *>(static_cast<const char *>(p) + so); };
    WD_HIP(wd::launch_force_links(static_cast<char *>(P) + po, at(x_e), at(z_o), at(y_e), at(w_o),
                                  static_cast<const char *>(UR64) + (size_t)8 * ctx->d * ctx->d * ctx->spre[l] * el,
                                  U ? static_cast<const char *>(U) + po : nullptr, ctx->g[l], ctx->N, ctx->rep, scale,
                                  accumulate, st));
  }
  WD_HIP(hipStreamSynchronize(st));
  return WDIRAC_OK;
}

// ------------------------------------------------------------ clover force
static size_t clover_offset(const wdirac_ctx *c, int l) {
  return (size_t)4 * c->d * (2 * c->d + 1) * c->spre[l] * 2 * 8;
}

static int clover_force_checks(const wdirac_ctx *ctx, const void *P, const void *U, const void *clov64, double m0,
                               double csw, int exponential, int gradient, int accumulate, const void *workspace) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(P, "out"));
  WD_TRY(check_ptr(U, "U"));
  WD_TRY(check_ptr(clov64, "clov64"));
  WD_TRY(check_ptr(workspace, "workspace"));
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  if (!std::isfinite(m0) || !std::isfinite(csw) || 4.0 + m0 == 0.0)
    return fail(WDIRAC_EINVAL, "m0 and csw must be finite and 4 + m0 != 0");
  if (exponential != 0 && exponential != 1) return fail(WDIRAC_EINVAL, "exponential must be 0 or 1");
  if (gradient != 0 && gradient != 1) return fail(WDIRAC_EINVAL, "gradient must be 0 or 1");
  if (accumulate != 0 && accumulate != 1) return fail(WDIRAC_EINVAL, "accumulate must be 0 or 1");
  return WDIRAC_OK;
}

int wdirac_force_eo_clover(const wdirac_ctx *ctx, void *P, const void *x_e, const void *UR64, const void *U,
                           const void *clov64, double m0, double csw, int exponential, double scale, int gradient,
                           int accumulate, void *workspace, void *stream) {
  WD_TRY(clover_force_checks(ctx, P, U, clov64, m0, csw, exponential, gradient, accumulate, workspace));
  WD_TRY(check_ptr(x_e, "x_e"));
  WD_TRY(check_ptr(UR64, "UR64"));
  const hipStream_t st = S(stream);
  const CloverForceWs w = carve_clover_force(ctx, workspace);
  // z_o = D_oo^{-1} D_oe x;  y_e = D_ee x - D_eo z_o = D-hat x;  w_o = D_oo^{-1} D_eo^+ y_e
  const auto chop = [&](void *out, const void *in, int parity, int dagger, double beta, const void *cx) {
    return hop(ctx, out, in, UR64, parity, dagger, 1, 0.0, nullptr, beta, WDIRAC_F64, nullptr, st, nullptr, nullptr,
               nullptr, clov64, cx);
  };
  WD_TRY(chop(w.z_o, x_e, 1, 0, 1.0, nullptr));
  WD_TRY(chop(w.y_e, w.z_o, 0, 0, -1.0, x_e));
  WD_TRY(chop(w.w_o, w.y_e, 1, 1, 1.0, nullptr));
  const size_t el = ctx->real ? 8 : 16;
  for (int l = 0; l < ctx->nlat; ++l) {
    const size_t so = (size_t)4 * ctx->d * ctx->spre[l] * 16;
    const size_t po = links_offset(ctx, l);
    auto at = [so](const void *p) { return static_cast<const void *>(static_cast<const char *>(p) + so); };
    const char *Ul = static_cast<const char *>(U) + po;
    WD_HIP(wd::launch_force_links(static_cast<char *>(P) + po, at(x_e), at(w.z_o), at(w.y_e), at(w.w_o),
                                  static_cast<const char *>(UR64) + (size_t)8 * ctx->d * ctx->d * ctx->spre[l] * el,
                                  gradient ? Ul : nullptr, ctx->g[l], ctx->N, ctx->rep, scale, accumulate, st));
    WD_HIP(wd::launch_clover_force(static_cast<char *>(P) + po, at(x_e), at(w.z_o), at(w.y_e), at(w.w_o), Ul,
                                   static_cast<const char *>(clov64) + clover_offset(ctx, l), w.F, w.K, w.G, w.Us,
                                   ctx->g[l], ctx->N, ctx->rep, m0, csw, exponential, 0.0, csw / 8.0 * scale,
                                   gradient, 1, st));
  }
  WD_HIP(hipStreamSynchronize(st));
  return WDIRAC_OK;
}

int wdirac_force_clover_logdet(const wdirac_ctx *ctx, void *P, const void *U, const void *clov64, double m0,
                               double csw, int exponential, double scale, int gradient, int accumulate,
                               void *workspace, void *stream) {
  WD_TRY(clover_force_checks(ctx, P, U, clov64, m0, csw, exponential, gradient, accumulate, workspace));
  const hipStream_t st = S(stream);
  const CloverForceWs w = carve_clover_force(ctx, workspace);
  for (int l = 0; l < ctx->nlat; ++l) {
    const size_t po = links_offset(ctx, l);
    WD_HIP(wd::launch_clover_force(static_cast<char *>(P) + po, nullptr, nullptr, nullptr, nullptr,
                                   static_cast<const char *>(U) + po,
                                   static_cast<const char *>(clov64) + clover_offset(ctx, l), w.F, w.K, w.G, w.Us,
                                   ctx->g[l], ctx->N, ctx->rep, m0, csw, exponential, 1.0, csw / 8.0 * scale,
                                   gradient, accumulate, st));
  }
  WD_HIP(hipStreamSynchronize(st));
  return WDIRAC_OK;
}

int wdirac_clover_logdet(const wdirac_ctx *ctx, double *logdet, const void *clov64, void *workspace, void *stream) {
  WD_TRY(check_ctx(ctx));
  WD_TRY(check_ptr(logdet, "logdet"));
  WD_TRY(check_ptr(clov64, "clov64"));
  WD_TRY(check_ptr(workspace, "workspace"));
  if (!wd::clover_supported(ctx->d)) return fail(WDIRAC_EUNSUPPORTED, "clover term available for d_R in {2,3,4,6}");
  const hipStream_t st = S(stream);
  const CloverForceWs w = carve_clover_force(ctx, workspace);
  for (int l = 0; l < ctx->nlat; ++l) {
    WD_HIP(wd::launch_clover_logdet(static_cast<const char *>(clov64) + clover_offset(ctx, l), w.part, ctx->g[l],
                                    ctx->d, st));
    WD_TRY(reduce_to_host(&logdet[l], w.part, wd::clover_logdet_blocks(ctx->g[l]), w.dtmp, st));
  }
  return WDIRAC_OK;
}

}  // extern "C"
