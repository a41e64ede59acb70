// Host side of the 16-bit fits: slab plan, choice of the form, parameters and
// dispatch to the kernels of mls_fit_lp.h.
#include <math.h>
#include <string.h>

#include "../../include/mls.h"
#include "mls_fit_lp.h"

namespace mls {

// Slab plan: feature tiles per slab (1..8) and attributes per slab (at most
// kDsCap) that cover D with the fewest padded columns in total.
static_assert((8 * 16 - 1) / 1 >= MLS_LP_MAX_SLAB_CONSTANT && kDsCap == MLS_LP_MAX_SLAB_CONSTANT,
              "constant-basis slab limit");
static_assert((8 * 16 - 6) / 3 >= MLS_LP_MAX_SLAB_LINEAR && kDsCap == MLS_LP_MAX_SLAB_LINEAR,
              "linear-basis slab limit");
static_assert((8 * 16 - 15) / 6 == MLS_LP_MAX_SLAB_QUADRATIC, "quadratic-basis slab limit");

int lp_max_slab(int degree) {
  const int m = basis_terms(degree), nmom = moment_terms(degree);
  const int ds = (8 * 16 - nmom) / m;
  return ds < kDsCap ? ds : kDsCap;
}

void lp_slab_plan(int degree, int D, int forced_ds, int* nts_out, int* ds_out, int* nslab_out) {
  const int m = basis_terms(degree), nmom = moment_terms(degree);
  if (forced_ds > 0) {
    const int ds = forced_ds < D ? forced_ds : D;
    int nts = 1;
    while (nts * 16 < nmom + m * ds) ++nts;
    *nts_out = nts;
    *ds_out = ds;
    *nslab_out = (D + ds - 1) / ds;
    return;
  }
  int best_cost = 1 << 30, best_nts = 8, best_ds = 1, best_ns = D;
  for (int nts = 1; nts <= 8; ++nts) {
    int ds = (nts * 16 - nmom) / m;
    if (ds > kDsCap) ds = kDsCap;
    if (ds < 1) continue;
    const int dsu = ds < D ? ds : D;
    const int ns = (D + dsu - 1) / dsu;
    const int cost = ns * nts;
    if (cost < best_cost || (cost == best_cost && nts > best_nts)) {
      best_cost = cost;
      best_nts = nts;
      best_ds = dsu;
      best_ns = ns;
    }
  }
  // the smallest tile count that still holds best_ds attributes
  int nts = 1;
  while (nts * 16 < nmom + m * best_ds) ++nts;
  *nts_out = nts;
  *ds_out = best_ds;
  *nslab_out = best_ns;
}

// Slabs of the two-pass form: attribute tiles of 16, attributes per slab.
static void shape_slab_plan(int D, int* ntv, int* ds, int* nslab) {
  *nslab = (D + kShapeDsCap - 1) / kShapeDsCap;
  *ds = (D + *nslab - 1) / *nslab;
  *ntv = (*ds + 15) / 16;
}

// ---- served batches ----

bool lp_batch_class(const FitArgs& a, bool fp16, int terms, LPBatchClass* cls) {
  if (a.wkind != 0 || a.grads || a.rigid) return false;
  // batch kernels exist for each format's default term count
  if (terms != (fp16 ? 2 : 3)) return false;
  int nts, ds, nslab;
  if (lp_use_shape_form(a.degree, a.D, fp16, a.wkind, false, terms, 0, a.lp_form)) {
    shape_slab_plan(a.D, &nts, &ds, &nslab);
    nts += kBatchShape;
  } else {
    lp_slab_plan(a.degree, a.D, a.lp_slab, &nts, &ds, &nslab);
  }
  cls->deg = a.degree;
  cls->nts = nts;
  cls->terms = terms;
  cls->fp16 = fp16;
  const int64_t tiles = (int64_t)((a.W + kCols - 1) / kCols) * ((a.H + kRows - 1) / kRows);
  cls->blocks = tiles * nslab;
  return true;
}

size_t lp_params_bytes() { return sizeof(LPParams); }

// Parameters of a fit in either form over all points (launch_fit_lp and the
// served batches; two passes set their own slabs).
static LPParams dense_lp_params(const FitArgs& a, const float* vals_s, const float* shift,
                                const float* scale, bool fp16) {
  int nts, ds, nslab;
  lp_slab_plan(a.degree, a.D, a.lp_slab, &nts, &ds, &nslab);
  LPParams p{};
  p.pts = a.pts;
  p.vals = vals_s;
  p.shift = shift;
  p.scale = scale;
  p.n = a.n;
  p.D = a.D;
  p.Ds = ds;
  p.nslab = nslab;
  p.inv_hd = 1.0 / a.h;
  p.inv_h = (float)p.inv_hd;
  p.x0 = a.x0; p.y0 = a.y0; p.dx = a.dx; p.dy = a.dy;
  p.W = a.W; p.H = a.H;
  p.tiles_x = (a.W + kCols - 1) / kCols;
  p.tiles = p.tiles_x * ((a.H + kRows - 1) / kRows);
  p.tau = a.tau;
  p.floor_w = a.floor_w;
  // weight below exp(-64) ~ 1.6e-28 at every node of the tile: the tile
  // spans at most half its diagonal from the anchor
  const double sxd = a.dx / a.h, syd = a.dy / a.h;
  const double half = 0.5 * sqrt((double)(kCols * kCols) * sxd * sxd +
                                 (double)(kRows * kRows) * syd * syd);
  const double reach = 8.0 + half;
  p.cutoff2 = (float)(reach * reach);
  // float16: a weight of 2^-25 or less (times the 2^15 gain, r^2 >= 40 ln 2)
  // rounds to zero in both of its terms; 27.8 leaves 0.07 for the float32
  // exponent.  bfloat16 has float32's range: only the anchor test applies.
  p.reach2 = fp16 ? 27.8f : __builtin_inff();
  p.list_log = (float)(log((double)a.n) + 36.0 * 0.6931471805599453);
  p.fields = a.fields;
  p.deg_out = a.deg_out;
  p.grads = nullptr;
  p.torder = nullptr;
  p.tile_start = nullptr;
  p.tile_list = nullptr;
  return p;
}

void lp_params_write(const FitArgs& a, const float* vals_s, const float* shift,
                     const float* scale, bool fp16, void* out) {
  LPParams p = dense_lp_params(a, vals_s, shift, scale, fp16);
  int ntv;
  if (lp_use_shape_form(a.degree, a.D, fp16, a.wkind, false, fp16 ? 2 : 3, 0, a.lp_form))
    shape_slab_plan(a.D, &ntv, &p.Ds, &p.nslab);
  memcpy(out, &p, sizeof(p));
}

hipError_t launch_fit_lp_batch(const LPBatchClass& c, const void* d_params, const uint32_t* d_items,
                               int n_items, const uint32_t* d_total, uint32_t* d_head,
                               uint32_t* d_done, uint32_t* d_skipped, uint32_t* h_complete,
                               const uint32_t* h_cancel, int grid, hipStream_t s) {
  LPBatch b;
  b.reqs = (const LPParams*)d_params;
  b.items = (const uint2*)d_items;
  b.total = d_total;
  b.head = d_head;
  b.done = d_done;
  b.skipped = d_skipped;
  b.complete = h_complete;
  b.cancel = h_cancel;
  b.n_items = n_items;
  if (c.terms != (c.fp16 ? 2 : 3)) return hipErrorInvalidValue;
  return c.fp16 ? launch_batch_fp16(b, c.deg, c.nts, grid, s)
                : launch_batch_bf16(b, c.deg, c.nts, grid, s);
}

// Largest node offset across a tile, in units of h.
double lp_tile_extent(double dx, double dy, double h) {
  const double ex = (double)(kCols - 1) * fabs(dx / h), ey = (double)(kRows - 1) * fabs(dy / h);
  return ex > ey ? ex : ey;
}

bool lp_use_shape_form(int degree, int D, bool fp16, int wkind, bool grads, int terms,
                       int forced_ds, int form) {
  if (wkind != 0 || grads || degree < 1) return false;
  // two passes carry an attribute in two terms, which float16 callers can ask
  // more than (bfloat16's default is three, and two passes its plan since they
  // exist)
  if (fp16 && terms > kShapeS2) return false;
  if (form == 1) return false;
  if (form == 2) return true;
  // The library's choice.  Two passes list once and contract twice; each has
  // a chunk's weights, tables and barrier, so fewer matrix instructions alone
  // do not pay.  float16 (7,351 points, 701 x 643, us one pass / two): one slab
  // either way, quadratic d = 5 346 / 491, linear d = 33 465 / 592; two slabs
  // in one pass, quadratic d = 19 687 / 554, linear d = 48 729 / 621, d = 64
  // 869 / 709: two passes where they need fewer slabs.  bfloat16, whose third
  // term costs one pass more, also where one pass issues 2.4 times the matrix
  // instructions: linear d = 19 (2.27 times) 522 / 617, d = 33 (2.5) 741 / 707,
  // quadratic d = 15, 3,000 points (4.4) 456 / 353.
  int nts, ds, nslab;
  lp_slab_plan(degree, D, forced_ds, &nts, &ds, &nslab);
  const int nslab2 = (D + kShapeDsCap - 1) / kShapeDsCap;
  if (fp16) return nslab > nslab2;
  const int one = nslab * nts * (2 * terms - 1);
  const int per2 = (D + nslab2 - 1) / nslab2;
  const int two = nslab2 * ((2 * terms - 1) + 3 * ((per2 + 15) / 16));
  return 5 * one >= 12 * two;
}

hipError_t launch_fit_lp(const FitArgs& a, const float* vals_s, const float* shift,
                         const float* scale, bool fp16, int terms, const LPCells* cells,
                         hipStream_t stream) {
  // the form depends on the request, not on the slab width (a tuning knob
  // that must not change a result bit)
  if (lp_use_shape_form(a.degree, a.D, fp16, a.wkind, a.grads != nullptr, terms, 0,
                        a.lp_form)) {
    LPParams p = dense_lp_params(a, vals_s, shift, scale, fp16);
    int ntv;
    shape_slab_plan(a.D, &ntv, &p.Ds, &p.nslab);
    return fp16 ? launch_shape_fp16(p, a.degree, ntv, terms, stream)
                : launch_shape_bf16(p, a.degree, ntv, terms, stream);
  }
  // the same parameters a served batch passes for the request, so that a
  // request computes the same bits alone and in a batch
  int nts, ds, nslab;
  lp_slab_plan(a.degree, a.D, a.lp_slab, &nts, &ds, &nslab);
  LPParams p = dense_lp_params(a, vals_s, shift, scale, fp16);
  p.grads = a.grads;
  const bool wend = a.wkind == 1;
  if (wend) {
    if (!cells) return hipErrorInvalidValue;
    p.pts = cells->pts_s;
    p.vals = cells->vals_ts;
    p.torder = cells->torder;
    p.slots = (int)tile_order_slots(p.tiles_x, p.tiles / p.tiles_x);
    p.tile_start = cells->tile_start;
    p.tile_list = cells->tile_list;
    return fp16 ? launch_lp_wend_fp16(p, a.degree, nts, terms, stream)
                : launch_lp_wend_bf16(p, a.degree, nts, terms, stream);
  }
  return fp16 ? launch_lp_fp16(p, a.degree, nts, terms, stream)
              : launch_lp_bf16(p, a.degree, nts, terms, stream);
}

}  // namespace mls
