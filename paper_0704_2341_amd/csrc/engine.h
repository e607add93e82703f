// Host-side engine: kernel launchers and handle structures.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "common.h"

namespace grg {

constexpr int kMaxRhs = 16;
// hop schedule of the hop-per-wavefront form of every stencil (64 sites of one
// RHS per item, a workgroup of eight wavefronts)
constexpr int kSplitForm = 8, kSplitSites = 64;
constexpr int kMaxGridValue = 4096;  // largest stencil/BLAS grid (sizes partial sums)

void set_error(const char *fmt, ...);

#define GRG_TRY_HIP(expr)                                                                    \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) {                                                              \
            ::grg::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, \
                             __LINE__);                                                      \
            return GRG_EHIP;                                                                 \
        }                                                                                    \
    } while (0)

#define GRG_TRY(expr)                        \
    do {                                     \
        grg_status s_ = (expr);              \
        if (s_ != GRG_OK) return s_;         \
    } while (0)

// ------------------------------------------------------------------ kernels
struct DslashArgs {
    const void *in;
    void *out;
    const void *U;
    const uint8_t *mask;  // output-site mask, nullptr = every site
    int sel;              // rows kept: mask[s] == sel
    double diag;          // 4 + m0
    Geom g;
    int nrhs;
    int SB;               // sites per work item == workgroup size
    int RG;               // right-hand sides per work item
    int split;            // 1: one hop per loop iteration, 0: one direction (two hops)
    int chunk;            // items per XCD chunk (0 = one contiguous eighth per XCD)
    int march;            // > 0: t-marching kernel with time chunks of this length
                          //      (64 sites x RG RHS wavefronts per workgroup)
    double *partials;     // [nrhs][3][grid] or nullptr
    const void *dot_with; // the fused dots use this field instead of `in` (or nullptr)
    int out_canon = 0;    // out is a canonical complex128 field (site-parallel forms, no sums)
    const uint8_t *in_mask = nullptr;  // canonical hop-per-wavefront form only: in is read on the
    int in_sel = 0;                    // sites with in_mask[s] == in_sel (nullptr: on every site)
};

// Stencil between the compact parity halves of the even-odd reduction
// (kernels_eo.hip): out = alpha in2 + beta (H in) on the rest sites of parity
// po, H the hopping term (D minus its diagonal).
struct EoArgs {
    const void *in;       // compact field of parity 1 - po
    const void *in2;      // compact field of parity po, or nullptr (alpha term dropped)
    void *out;            // compact field of parity po
    const void *U;        // links, [2][compact tiles][4][9][64]
    const uint8_t *mask;  // [2][Vhs]: 1 on coarse sites and padding
    int po;               // output parity
    double alpha, beta;
    Geom g;               // the full lattice
    int Vh, Vhs;          // half volume, and padded to whole tiles (multiple of 256)
    int nrhs, SB, RG, hops, chunk;
    int march;            // hops == 3: time slices per workgroup item (t-marching form)
    double *partials;     // [nrhs][3][grid] or nullptr
    const void *dot_with; // parity po, or nullptr: the sums are |out|^2 only (re, im zero)
    const int *active;    // per RHS: 0 writes zero for that RHS (nullptr: all active)
    // full-layout variants (the first and last steps of a reduced solve read
    // and write the unreduced fields directly): in / in2 indexed by the full
    // site; out written to the full field, together with the same-index site
    // of the other parity, copied from `partner` (compact, parity 1 - po)
    int in_full, in2_full, out_full;
    const void *partner;
};

// out = u + sigma (x + sum_j f[j][rhs] e_j) in FP64 (u, x nullable): the
// defect correction's iterate from its kept corrections e_j (inner precision)
constexpr int kCorrPool = 16;
struct CombineArgs {
    const void *e[kCorrPool];
    const double *f;      // [kCorrPool][kMaxRhs]
    int n;                // corrections in use
    const void *u, *x;    // FP64 or nullptr
    void *out;            // FP64, may alias x or u
    double sigma;
};

// A tuned launch of the stencil for one precision and RHS count.
struct DslashTune {
    int valid = 0;
    int SB = 128, RG = 1, split = 0, grid = 0, chunk = 0, march = 0;
    float ms = 0;
};

struct CoarseArgs {
    const void *in;       // internal FP64 lattice field
    void *out;            // canonical coarse [nrhs][nb][12] complex128
    const void *U;        // internal FP64 links
    const int32_t *q;     // coarse index -> site
    int nb;
    double diag;
    Geom g;
    int nrhs;
};

// Fused FP64 defect-correction step (see dc_update_kernel).
struct DcArgs {
    const void *e;        // inner solution, internal tiles in the inner precision
    const void *U;        // FP64 links
    const void *r_in;     // FP64 residual before the step
    const void *x_in;     // FP64 iterate before the step, or nullptr for zero
    void *r_out, *x_out;  // FP64 results (may alias the inputs)
    const double *f;      // per-RHS factor of e (the inner right-hand side was r / f)
    void *r_next;         // r_out * s_next in the inner precision (next inner rhs), or nullptr
    const double *s_next; // per-RHS scale of r_next
    const uint8_t *mask;  // 1 on coarse sites
    double diag;          // 4 + m0
    Geom g;
    int nrhs;
    double *partials;     // [nrhs][grid]: |r_out|^2
    int RG, chunk, march; // t-marching launch (march > 0), as in DslashArgs
    int split = 0;        // kSplitForm: the hop-per-wavefront form
    int ring;             // with march > 0 and BF16 e: the LDS-ring form of the t-marching step
    int grp_first;        // ring form: work items ordered with the RHS group fastest, so the
                          // groups of one tile run together on one XCD and share its links
    int r_in32 = 0;       // r_in is stored in FP32 (float2 per complex), else FP64
    int r_out32 = 0;      // r_out is stored in FP32 (rounded from the FP64 result), else FP64
    // r_next in the compact even-odd halves (the reduced solve's right-hand
    // side) instead of the full layout: the half of parity next_par first, the
    // other next_half elements on (0: full layout)
    size_t next_half = 0;
    int next_par = 0;
};

hipError_t launch_dslash(int prec, const DslashArgs &a, int grid, hipStream_t st);
// SB: workgroup of the site-parallel kernel (a.march == 0); with a.march > 0
// the t-marching kernel runs with 64 * a.RG threads per workgroup (a.ring: its
// LDS-ring form, BF16 e only, 64 sites per x-y-z tile made of whole x-rows).
hipError_t launch_dc_update(int prec, const DcArgs &a, int grid, int SB, hipStream_t st);
// The hop-per-wavefront forms (kernels_split.hip): 512 threads, one RHS per
// item.  canonical (no sums): in and out are canonical complex128 fields that
// do not overlap.
hipError_t launch_dslash_split(int prec, const DslashArgs &a, bool canonical, int grid, hipStream_t st);
// The t-march over canonical fields (kernels_ring.hip): every row, no sums, in and
// out canonical complex128 fields that do not overlap; a.march slices per item,
// grid (workgroups of one wavefront) a multiple of 8.
hipError_t launch_canon_march(int prec, const DslashArgs &a, int grid, hipStream_t st);
hipError_t launch_eo_split(int prec, const EoArgs &a, int grid, hipStream_t st);
hipError_t launch_dc_split(int prec, const DcArgs &a, int grid, hipStream_t st);
hipError_t launch_dslash_coarse(const CoarseArgs &a, hipStream_t st);
// b = D_rb x_b from the canonical coarse vector (kernels_coarse.hip): internal
// FP64 field, zero on the coarse sites
// With partials set, also the per-workgroup |b|^2 per RHS ([nrhs][rb_apply_grid(g)]).
// With pair set, b also in precision pair_prec as a compact even-odd pair
// (parity `first` at compact index s / 2, the other parity `half` elements on).
hipError_t launch_rb_apply(const Geom &g, const double *xb, const int32_t *bidx, int nb, const void *U64,
                           void *out, int nrhs, hipStream_t st, double *partials = nullptr,
                           int pair_prec = -1, void *pair = nullptr, size_t half = 0, int first = 0);
int rb_apply_grid(const Geom &g);
// y_b = [D (u + sigma sum_j f_j e_j)]_b, u = x_b on the coarse sites, from the
// kept corrections (inner precision prec) at the coarse sites' neighbours
hipError_t launch_coarse_combine_apply(int prec, const Geom &g, const double *xb, const int32_t *qsites,
                                       const int32_t *bidx, int nb, const void *U64, double diag,
                                       const CombineArgs &a, double *yb, int nrhs, hipStream_t st,
                                       bool adjacent);
hipError_t launch_eo_hop(int prec, const EoArgs &a, int grid, hipStream_t st);
// compact field of parity par <-> full field (zero off that parity)
hipError_t launch_eo_scatter(int prec, const Geom &g, int nrhs, int par, const void *src, void *dst,
                             bool to_full, hipStream_t st);
hipError_t launch_eo_pack_links(int prec, const Geom &g, int Vhs, const void *U, void *Ueo, hipStream_t st);
hipError_t launch_eo_pack_mask(const Geom &g, int Vhs, const uint8_t *mask, uint8_t *meo, hipStream_t st);
hipError_t launch_pack_gauge(const double *src, const Geom &g, const int bc[4], void *u64,
                             void *u32, void *u16, hipStream_t st);
hipError_t launch_pack_spinor(int prec, const double *src, void *dst, const Geom &g, int nrhs,
                              hipStream_t st, const uint8_t *mask = nullptr, int keep = 0);
hipError_t launch_unpack_spinor(int prec, const void *src, double *dst, const Geom &g, int nrhs,
                                hipStream_t st);
hipError_t launch_scatter_coarse(const double *xb, void *dst, const int32_t *bidx, int nb,
                                 const Geom &g, int nrhs, hipStream_t st);

// BLAS-1 on internal fields.  Every kernel walks sites in work items of
// SB sites x all RHS (looped); partial sums go to [nrhs][k][grid] doubles.
struct BlasShape {
    Geom g;
    int nrhs;
    int grid;   // workgroups, multiple of 8
    int half = 0;  // a compact parity half (hidx) instead of a full field (fidx)
};

// partials -> per-RHS reductions (fixed-order tree, deterministic)
//  mode kAlpha: in k = 3 (re<q,r>, im<q,r>, |q|^2); alpha[r] = <q,r>/|q|^2 if
//               active[r], else 0.  Also stores |q|^2 in aux[r].
//  mode kNorm : in k = 1; out2[r] = sum; active[r] = sum > thr2[r].
//  mode kNorm3: as kNorm from the third of k = 3 sums (a stencil's fused |out|^2).
//  part (kNorm, kNorm3; optional): part[r] = thr2[r] finite (the RHS takes
//  part in the solve; an infinite threshold marks one that does not).
enum { kAlpha = 0, kNorm = 1, kNorm3 = 2 };
// Where a reduction also leaves RHS r's |.|^2 for the host: pinned words 2r and
// 2r + 1, each with tag above and half the value's bits below.  An 8-byte store is
// whole, so a host that sees the tag in both words has the value without waiting
// for the stream (27 us from enqueueing five short launches and a read to having
// it, 20 so).
struct HostNorms {
    unsigned long long *words = nullptr;
    unsigned tag = 0;
};
hipError_t launch_reduce(int mode, const double *partials, int nparts, int nrhs, double2 *alpha,
                         double *out2, const double *thr2, int *active, hipStream_t st,
                         int *part = nullptr, const HostNorms &host = HostNorms());

// Scalars taken straight from per-workgroup partials by the vector kernels,
// instead of by a reduction launch between: for as few rows as kFoldRows.  A
// reduction of few rows is a launch of 2.6-5 us that the next kernel waits for;
// summing them again in every wavefront adds about 1 us to that kernel (S_bb at
// 8^4, BF16: 897 -> 814 us, the V-cycle 18.4 -> 15.4 ms; with 948 rows the
// BiCGstab solve gains nothing, 1771 against 1800 us).
constexpr int kFoldRows = 512;
struct FoldMr {
    const double *dot = nullptr;  // the stencil's sums [nrhs][3][ndot]; nullptr: alpha is given
    int ndot = 0;
    const double *nrm = nullptr;  // |r|^2 before this step [nrhs][nnrm] (nullptr: active alone decides)
    int nnrm = 0;
    const double *thr2 = nullptr; // with nrm: a RHS at or below it takes no step
    const int *active = nullptr;
};
// One x update for two minimal-residual steps (p = r, alpha given): with r_out the
// step leaves x alone and writes its new r there; the next one, given that
// step's r and alpha as r_prev and alpha_prev, updates x with both.
struct MrLazy {
    void *r_out = nullptr;
    const void *r_prev = nullptr;
    const double2 *alpha_prev = nullptr;
};
enum MrX { kMrXAdd, kMrXZero, kMrXLater, kMrXPair, kMrXPairZero };
// x += alpha r ; r -= alpha q ; partial |r|^2     (one MR/GCR step; x_zero:
// x is taken as zero and not read, the first step from x = 0)
hipError_t launch_mr_update(int prec, const BlasShape &sh, void *x, void *r, const void *q,
                            const void *p, const double2 *alpha, double *partials,
                            hipStream_t st, bool x_zero = false, const FoldMr &fold = FoldMr(),
                            const MrLazy &lazy = MrLazy());
// partial |v|^2
hipError_t launch_norm2(int prec, const BlasShape &sh, const void *v, double *partials,
                        hipStream_t st);
// r = b - ax (FP64), partial |r|^2
hipError_t launch_sub_norm(const BlasShape &sh, const void *b, const void *ax, void *r,
                           double *partials, hipStream_t st);
// y (prec_out) = beta*y + scale[r] * x (prec_in); scale from a device array
// of per-RHS reals, multiplied by 1/sqrt(scale) when inv_sqrt != 0.  With
// y_half > 0, y is a compact even-odd pair (parity y_first's half first, the
// other y_half elements on; beta 0).
hipError_t launch_axpy_convert(int prec_in, int prec_out, const BlasShape &sh, const void *x,
                               void *y, const double *scale, int inv_sqrt, int beta,
                               const int *active, hipStream_t st, size_t y_half = 0, int y_first = 0);
// y = x - y (FP64), used for u - z
hipError_t launch_xmy(const BlasShape &sh, const void *x, void *y, hipStream_t st);
hipError_t launch_combine(int prec, const BlasShape &sh, const CombineArgs &a, hipStream_t st);
// Schur complement approximations of section 3 on the boundary, the rest
// sites next to a coarse site (kernels_approx.hip).  site: the boundary's sites
// in lattice order, map: site -> index in it, or negative; count: scratch of
// boundary_blocks ints; info[0]: the boundary sites' number, info[1]: the stamp
// of the rows with which a boundary site has a neighbour whose t is not zero.
struct ApproxArgs {
    Geom g;
    const double *xb;     // canonical coarse vector
    double *yb;
    const int32_t *q, *bidx;
    int nb;
    const int32_t *site, *map;
    int nbnd;             // the boundary sites' number, or with info set at least that
    const void *U;        // FP64 links
    const void *rows;     // row sums of D_rr (one FP64 field), nullptr: couplings inside D_rr ignored
    int linked;           // a boundary site has, or may have, a neighbour whose t is not zero
    double diag;          // 4 + m0
    void *t, *p;          // compact FP64 fields over the boundary, internal tiles
    int nrhs;
    // info set: what the host does not know yet.  launch_boundary_coarse leaves
    // host[0] = info[0] + 1 and, with stamp > 0 the rows' one, host[1] = stamp or
    // -stamp, as such a neighbour exists or not (pinned words, each whole).
    const int *info;
    int *host, stamp;
};
int boundary_blocks(const Geom &g);
hipError_t launch_boundary_build(const Geom &g, const int32_t *bidx, int *count, int32_t *site, int32_t *map,
                                 int *info, hipStream_t st);
hipError_t launch_boundary_rows(const Geom &g, const int32_t *bidx, const void *U, double diag, void *rows,
                                int32_t *map, int *info, int stamp, hipStream_t st);
hipError_t launch_boundary_source(const ApproxArgs &a, hipStream_t st);
hipError_t launch_boundary_apply(const ApproxArgs &a, hipStream_t st);
hipError_t launch_boundary_coarse(const ApproxArgs &a, hipStream_t st);
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t st);
hipError_t launch_copy(int prec, const BlasShape &sh, const void *x, void *y, hipStream_t st);

// BiCGstab vector steps and scalar reductions (kernels_blas.hip); sc holds
// rho, alpha, omega, beta per RHS as double2[4][kMaxRhs]:
//   kBicgS   s = r - alpha v               (r := s, a := r, b := v)
//   kBicgUpd x += alpha p + omega s, r = s - omega t, partials <r0, r>, |r|^2
//            (x, r, a := p, b := s, c := t, d := r0)
//   kBicgP   p = r + beta (p - omega v)    (r := p, a := r, b := v)
// and reductions kBicgInit (rho = |r0|^2), kBicgAlpha (alpha = rho / <r0, v>
// from the stencil's fused sums against r0), kBicgBeta (beta, rho, |r|^2).
enum { kBicgS = 0, kBicgUpd = 1, kBicgP = 2 };
enum { kBicgInit = 0, kBicgAlpha = 1, kBicgBeta = 2 };
// With fold.rows set, the step's own scalar comes from those partials (kBicgS:
// alpha from the stencil's sums; kBicgUpd: omega from the stencil's; kBicgP:
// beta, rho, |r|^2 and the active flags from kBicgUpd's) and the wavefront of
// each RHS's first unit writes it out: alpha and omega to sc, and rho, the
// flags and |r|^2 to the fold's outputs, which this launch does not read.
struct FoldBicg {
    const double *rows = nullptr;
    int n = 0;
    const double2 *rho = nullptr;  // current rho
    double2 *rho_out = nullptr;    // kBicgP
    const int *active = nullptr;
    int *active_out = nullptr;     // kBicgP
    const double *thr2 = nullptr;  // kBicgP
    double *rn2 = nullptr;         // kBicgP
    HostNorms host;                // kBicgP: with rn2
};
hipError_t launch_bicg(int prec, int mode, const BlasShape &sh, void *x, void *r, const void *a,
                       const void *b, const void *c, const void *d, double2 *sc,
                       double *partials, hipStream_t st, const FoldBicg &fold = FoldBicg());
hipError_t launch_bicg_reduce(int mode, const double *partials, int nparts, int nrhs, double2 *sc,
                              double *out2, const double *thr2, int *active, hipStream_t st,
                              const HostNorms &host = HostNorms());

// V-cycle (kernels_vcycle.hip): blocked links of the next level, restriction
// to / prolongation from the coarse sites (canonical fields), and linear
// combinations and dot products of canonical FP64 fields.
struct VcCoef {
    int n;                     // inputs in use, 1..3
    double2 c[3][kMaxRhs];     // per input and RHS
};
hipError_t launch_vc_block_links(const Geom &gf, const void *U64, const Geom &gc, double *out, hipStream_t st);
hipError_t launch_vc_restrict(const double *f, const double *t, double *coarse, const int32_t *q, int nb, int V,
                              int nrhs, hipStream_t st);
hipError_t launch_vc_prolong(const double *coarse, double *full, const int32_t *bidx, int nb, int V, int nrhs,
                             hipStream_t st);
hipError_t launch_vc_lincomb(size_t len, int nrhs, const VcCoef &cf, double *out, const double *in0,
                             const double *in1, const double *in2, hipStream_t st);
// A whole BiCGstab solve A x = f, x from zero, A = c D (mask == nullptr) or
// c D_rr on the sites with mask 0 (f read and x written there, x zero elsewhere),
// a workgroup per RHS (kernels_small.hip).  Lattices of at most kSmallSites
// sites; canonical FP64 fields, x not overlapping f.  Per RHS until
// |r| <= tol |f| or max_iter; with check > 0 the residual is then recomputed from
// x, the solve goes on if that misses tol (check times at most), and x = 0 is kept
// if x is no better.
// flags[0] is set if an RHS did not reach tol, flags[1] if a residual is not
// finite.
constexpr int kSmallSites = 256;
constexpr int kSmallIters = 20000;  // most iterations of one launch (which nothing interrupts): 0.5 s
struct SmallArgs {
    Geom g;
    const void *U;  // internal FP64 links
    const uint8_t *mask;
    double diag, c, tol;
    int max_iter, check;
    const double *f;
    double *x;
    int *flags;
};
hipError_t launch_small_bicgstab(const SmallArgs &a, int nrhs, hipStream_t st);
int vc_dot_grid(size_t len);
hipError_t launch_vc_dot(size_t len, int nrhs, const double *a, const double *b, double *partials,
                         hipStream_t st);

// GCR(m > 1): <q_j, q> for j < k, then q -= sum beta_j q_j, p -= sum beta_j p_j
// with beta_j = <q_j, q>/|q_j|^2, fused with the partials of
// (re<q,r>, im<q,r>, |q|^2) for the step length.
hipError_t launch_multidot(int prec, const BlasShape &sh, const void *Q, int k, const void *q,
                           double *partials, hipStream_t st);
hipError_t launch_reduce_multi(const double *partials, int nparts, int nrhs, int k,
                               const double *qnorm2, const int *active, double2 *beta,
                               hipStream_t st);
hipError_t launch_orthogonalise(int prec, const BlasShape &sh, const void *Q, const void *P,
                                int k, const double2 *beta, void *q, void *p, const void *r,
                                double *partials, hipStream_t st);

}  // namespace grg
