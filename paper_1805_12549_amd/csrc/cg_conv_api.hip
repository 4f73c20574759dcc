// Host side of the C ABI: argument validation, threshold folding (merged gate of
// Sec. 3.2 of the channel-gating paper), layout of the caller's `packed` buffer,
// kernel-family choice and launch sequencing.  No device memory is allocated here.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "cg_internal.h"
#include "point_piece.h"

namespace {

thread_local std::string g_err = "";

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
}  // namespace

namespace cg {
// records the calling thread's error text for cg_last_error(); returns `code`
int set_error(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int cu_count() {
  static std::atomic<int> cached[64];
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0) {
    if (dev < 64) n = cached[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) {
      if (dev < 64) cached[dev].store(n, std::memory_order_relaxed);
      return n;
    }
  }
  (void)hipGetLastError();
  return 256;
}

hipError_t allow_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
  return e;
}
}  // namespace cg

namespace {

int elem_bytes(int dtype) {
  switch (dtype) {
    case CG_F32: return 4;
    case CG_BF16: return 2;
    case CG_I8: return 1;
    case CG_I32: return 4;
    default: return 0;
  }
}

constexpr int kTables = 8;  // per-channel tables of 4-byte entries at the start of `packed`

struct Layout {
  size_t table_stride;   // bytes per table
  size_t w_base_off, w_base_bytes;
  size_t w_cond_off, w_cond_bytes;
  size_t wpk_base_off, wpk_cond_off;       // prepacked weights of the tiled kernel, if one covers the layer
  size_t wpd_base_off, wpd_cond_off;       // prepacked weights of the small-tile kernel, if it may be picked
  size_t wpt_base_off;                     // prepacked weights of the large-tile kernel beside the row-tiled one's (tile_too)
  size_t total;
};

}  // namespace

namespace {

enum Kernel { kNaive, kRows, kTile, kDirect };

// What one batch size runs on.
struct CallPlan {
  int n;
  Kernel kernel;
  cg::RowsPlan rows, rows_over;          // rows_over: for an output written over its residual
  cg::TilePlan tile;
  cg::DirectPlan direct, direct_rest;    // for `piece` images at a time and for what is left (none where piece divides n)
  int piece;
};

}  // namespace

struct cg_conv {
  cg_conv_desc d;           // copy of the descriptor (host pointers are dead after create)
  int ho, wo, c_cond;
  int variant;              // resolved CG_VARIANT_*: the kernel family that covers the shape
  bool direct_ok;           // the small-tile kernel's weights are packed too: it takes the layer, if not every batch of it
  bool point_ok;            // a 1x1 layer of the large-tile family that runs on the row-tiled kernel
  bool tile_too;            // ... and on the large-tile kernel where that suits the batch
  CallPlan first;           // plan for n_max
  Layout lay;
  cg::Params base;          // what is the same in every call
  std::vector<uint32_t> staging;  // host image of the tables; kept alive for the async copy
  // plans of other batch sizes, made on first use (7 us of host time) and kept, the last kKept of them
  static constexpr int kKept = 64;
  mutable std::mutex lock;
  mutable int kept_n[kKept] = {};          // their batch sizes; 0: none yet
  mutable int kept_next = 0;
  mutable std::vector<CallPlan> kept;      // (room for kKept from the start: a forward call allocates nothing)
};

namespace {

// Pure checks; no HIP call.  Fills geometry on success.
int validate(const cg_conv_desc* d, int* ho, int* wo) {
  if (!d) return fail(CG_EINVAL, "descriptor is NULL");
  if (d->struct_size != sizeof(cg_conv_desc))
    return fail(CG_EINVAL, "struct_size %u does not match this library's %zu", d->struct_size, sizeof(cg_conv_desc));
  if (d->n_max <= 0 || d->h <= 0 || d->w <= 0 || d->c_in <= 0 || d->c_out <= 0)
    return fail(CG_EINVAL, "n_max, h, w, c_in, c_out must be positive");
  if (d->stride < 1 || d->pad < 0) return fail(CG_EINVAL, "stride must be >= 1 and pad >= 0");
  if (d->kh <= 0 || d->kw <= 0) return fail(CG_EINVAL, "kernel size must be positive");
  if (!((d->kh == 3 && d->kw == 3) || (d->kh == 1 && d->kw == 1)))
    return fail(CG_EUNSUPPORTED, "kernel size %dx%d: only 3x3 and 1x1 are supported", d->kh, d->kw);
  if (d->pad >= d->kh && d->pad > 0) return fail(CG_EINVAL, "pad %d must be smaller than the kernel size", d->pad);
  if (d->c_base <= 0 || d->c_base > d->c_in) return fail(CG_EINVAL, "c_base must lie in (0, c_in]");
  if (d->groups < 0) return fail(CG_EINVAL, "groups must be >= 0");
  if (d->groups > 1) {
    if ((long long)d->c_base * d->groups != d->c_in)
      return fail(CG_EINVAL, "channel grouping needs c_base * groups == c_in (%d * %d != %d)", d->c_base, d->groups,
                  d->c_in);
    if (d->c_out % d->groups) return fail(CG_EINVAL, "channel grouping needs groups to divide c_out");
  }
  if (d->shuffle != 0 && d->shuffle != 1) return fail(CG_EINVAL, "shuffle must be 0 or 1");
  if (d->shuffle && d->groups <= 1) return fail(CG_EINVAL, "shuffle needs channel grouping (groups > 1)");
  if (!(d->tau_c >= 0.0f) || std::isinf(d->tau_c)) return fail(CG_EINVAL, "tau_c must be finite and >= 0");
  if (d->tile_hint < 0 || d->tile_hint >= (1 << 12)) return fail(CG_EINVAL, "tile_hint has bits outside its three fields");
  if (d->in_dtype != CG_F32 && d->in_dtype != CG_BF16 && d->in_dtype != CG_I8)
    return fail(CG_EINVAL, "in_dtype must be CG_F32, CG_BF16 or CG_I8");
  if (d->in_dtype == CG_I8) {
    if (d->delta_hi) return fail(CG_EUNSUPPORTED, "the upper gate threshold (delta_hi) exists for float inputs only");
    if (d->out_dtype != CG_I32 && d->out_dtype != CG_I8)
      return fail(CG_EINVAL, "int8 inputs need out_dtype CG_I32 or CG_I8");
    if (d->rq_shift < 0 || d->rq_shift > 31) return fail(CG_EINVAL, "rq_shift must lie in [0, 31]");
  } else if (d->out_dtype != CG_F32 && d->out_dtype != CG_BF16) {
    return fail(CG_EINVAL, "float inputs need out_dtype CG_F32 or CG_BF16");
  }
  if (d->epilogue & ~(CG_EPI_RELU | CG_EPI_AFFINE | CG_EPI_RESIDUAL)) return fail(CG_EINVAL, "unknown epilogue flag");
  if (d->variant != CG_VARIANT_AUTO && d->variant != CG_VARIANT_NAIVE && d->variant != CG_VARIANT_MFMA_ROWS &&
      d->variant != CG_VARIANT_TILE)
    return fail(CG_EINVAL, "unknown variant %d", d->variant);
  if (d->x_pixel_stride != 0 && d->x_pixel_stride < d->c_in)
    return fail(CG_EINVAL, "x_pixel_stride must be 0 or >= c_in");
  const int span_h = d->h + 2 * d->pad - d->kh, span_w = d->w + 2 * d->pad - d->kw;
  if (span_h < 0 || span_w < 0) return fail(CG_EINVAL, "kernel larger than the padded input");
  *ho = span_h / d->stride + 1;
  *wo = span_w / d->stride + 1;
  const long long m = (long long)d->n_max * *ho * *wo;
  if (m * (long long)d->c_out >= (1ll << 40)) return fail(CG_EUNSUPPORTED, "output too large");
  if (!d->w_base) return fail(CG_EINVAL, "w_base is NULL");
  const bool gated = d->c_base < d->c_in;
  if (gated && !d->w_cond) return fail(CG_EINVAL, "w_cond is NULL for a gated layer");
  if (gated) {
    if (d->in_dtype == CG_I8) {
      if (!d->gate_thr_i32) return fail(CG_EINVAL, "gate_thr_i32 is NULL for a gated int8 layer");
    } else {
      if (!d->gate_mean || !d->gate_var || !d->delta)
        return fail(CG_EINVAL, "gate_mean, gate_var and delta are required for a gated float layer");
      if (std::isnan(d->gate_eps)) return fail(CG_EINVAL, "gate_eps is NaN");
      for (int c = 0; c < d->c_out; ++c) {
        if (std::isnan(d->gate_mean[c]) || std::isnan(d->gate_var[c]) || std::isnan(d->delta[c]) ||
            (d->delta_hi && std::isnan(d->delta_hi[c])))
          return fail(CG_EINVAL, "NaN in the gate statistics of channel %d", c);
        if (std::isinf(d->gate_mean[c]) || std::isinf(d->gate_var[c]))
          return fail(CG_EINVAL, "infinite gate statistics in channel %d", c);
        if ((double)d->gate_var[c] + (double)d->gate_eps < 0.0)
          return fail(CG_EINVAL, "gate_var + gate_eps is negative in channel %d", c);
      }
    }
  }
  return CG_OK;
}

Layout make_layout(const cg_conv_desc& d, size_t wpk_base_bytes, size_t wpk_cond_bytes, size_t wpd_base_bytes,
                   size_t wpd_cond_bytes, size_t wpt_base_bytes) {
  Layout l{};
  const size_t eb = (size_t)elem_bytes(d.in_dtype);
  const size_t taps = (size_t)d.kh * d.kw;
  l.table_stride = align256((size_t)d.c_out * 4);
  size_t off = l.table_stride * kTables;
  l.w_base_bytes = (size_t)d.c_out * taps * d.c_base * eb;
  l.w_cond_bytes = (size_t)d.c_out * taps * (size_t)(d.c_in - d.c_base) * eb;
  l.w_base_off = off;
  off += align256(l.w_base_bytes);
  l.w_cond_off = off;
  off += align256(l.w_cond_bytes);
  l.wpk_base_off = off;
  off += align256(wpk_base_bytes);
  l.wpk_cond_off = off;
  off += align256(wpk_cond_bytes);
  l.wpd_base_off = off;
  off += align256(wpd_base_bytes);
  l.wpd_cond_off = off;
  off += align256(wpd_cond_bytes);
  l.wpt_base_off = off;
  off += align256(wpt_base_bytes);
  l.total = off;
  return l;
}

struct Plans {
  cg::RowsPlan v3;
  cg::TilePlan v4;
  cg::DirectPlan vd;
  int variant;
  bool direct_ok, point_ok, tile_too;
  size_t wpk_base_bytes, wpk_cond_bytes, wpd_base_bytes, wpd_cond_bytes, wpt_base_bytes;
};

int resolve_variant(const cg_conv_desc& d, Plans* pl) {
  pl->v4 = cg::tile_plan(d, cg::cu_count());
  pl->v3 = cg::rows_plan(d, cg::cu_count(), 0, 2);
  if (d.variant == CG_VARIANT_TILE && !pl->v4.ok)
    return fail(CG_EUNSUPPORTED, "the large-tile matrix-core kernel does not cover this shape/dtype");
  if (d.variant == CG_VARIANT_MFMA_ROWS && !pl->v3.ok)
    return fail(CG_EUNSUPPORTED, "the row-tiled matrix-core kernel does not cover this shape/dtype");
  int v = d.variant;
  if (v == CG_VARIANT_AUTO) v = pl->v3.ok ? CG_VARIANT_MFMA_ROWS : pl->v4.ok ? CG_VARIANT_TILE : CG_VARIANT_NAIVE;
  pl->variant = v;
  // 1x1 layers of stride 1 whose channel walk is whole stages run on the row-tiled kernel (unless a family was asked for by
  // name): 1024 channels at 14x14 x64, bf16 40 us against 99 on the large-tile kernel, int8 28 against 105
  pl->point_ok = false;
  if (d.variant == CG_VARIANT_AUTO && v != CG_VARIANT_MFMA_ROWS) {
    const cg::RowsPlan q = cg::point_plan(d, cg::cu_count());
    pl->point_ok = q.ok != 0;
    if (q.ok) pl->v3 = q;
  }
  pl->tile_too = pl->point_ok && pl->v4.ok && d.in_dtype == CG_BF16 && d.c_base == d.c_in && d.c_in >= 2048;    // (see pick_kernel)
  pl->vd = cg::direct_plan(d, 1, cg::cu_count());          // (what is packed does not depend on the batch)
  pl->direct_ok = d.variant == CG_VARIANT_AUTO && pl->vd.ok;      // (a family that was asked for by name is what runs)
  pl->wpd_base_bytes = pl->direct_ok ? pl->vd.wpk_bytes[0] : 0;
  pl->wpd_cond_bytes = pl->direct_ok ? pl->vd.wpk_bytes[1] : 0;
  const bool rows = v == CG_VARIANT_MFMA_ROWS || pl->point_ok;
  pl->wpk_base_bytes = rows ? pl->v3.wpk_base_bytes : v == CG_VARIANT_TILE ? pl->v4.wpk_base_bytes : 0;
  pl->wpk_cond_bytes = rows ? pl->v3.wpk_cond_bytes : v == CG_VARIANT_TILE ? pl->v4.wpk_cond_bytes : 0;
  pl->wpt_base_bytes = pl->tile_too ? pl->v4.wpk_base_bytes : 0;
  return CG_OK;
}

// The small-tile kernel's plan for a batch.  Its 32-bit offsets reach over 1 GiB of x and 2^30 pixels; where the plain kernel
// would be the other choice, a larger batch runs in pieces (of whole images: every pointer stays aligned as the pixels are).
// int8, 16 channels at 512x512, 300 images: 167 -> 9.0 ms.
void plan_direct(const cg_conv* h, int n, CallPlan* c) {
  c->direct = c->direct_rest = cg::DirectPlan{};
  c->piece = n;
  if (!h->direct_ok) return;
  c->direct = cg::direct_plan(h->d, n, cg::cu_count());
  if (c->direct.ok || h->variant != CG_VARIANT_NAIVE || h->point_ok) return;
  const long long limit = (1ll << 30) - 1, image = (long long)h->d.h * h->d.w * h->d.x_pixel_stride * elem_bytes(h->d.in_dtype);
  const long long px = (long long)h->ho * h->wo, piece = limit / (image > px ? image : px);
  if (piece < 1 || piece >= n) return;
  c->direct = cg::direct_plan(h->d, (int)piece, cg::cu_count());
  if (n % piece) c->direct_rest = cg::direct_plan(h->d, (int)(n % piece), cg::cu_count());
  if (n % piece && !c->direct_rest.ok) c->direct.ok = 0;
  c->piece = (int)piece;
}

// The kernel a batch runs on.  (Layers that neither tiled family covers: the small-tile kernel.)
void pick_kernel(const cg_conv* h, CallPlan* c) {
  c->kernel = h->variant == CG_VARIANT_MFMA_ROWS || h->point_ok ? kRows : h->variant == CG_VARIANT_TILE ? kTile : kNaive;
  // Dense bf16 1x1 layers with a deep K, which reads the operands of a product in larger pieces on the large-tile kernel: as
  // long as its tiles are whole rounds over the compute units, large-tile / row-tiled kernel, us: 4096 channels to 4096,
  // 8192 pixels 336 / 394, 2048 86 / 101; 2048 to 2048, 4096 pixels 51 / 58.  Rounds that are not: 4096 to 4096, 700
  // pixels 65 / 44; 2048 to 512, 12544 57 / 50.  At 1024 channels the two are equal.
  if (h->tile_too && c->tile.ok) {
    const int cu = cg::cu_count(), rounds = (c->tile.wgs + cu - 1) / cu;
    if ((long long)c->tile.wgs * 100 >= 97ll * rounds * cu) c->kernel = kTile;
  }
  if (!h->direct_ok || !c->direct.ok) return;
  if (c->kernel == kNaive) {
    c->kernel = kDirect;
    return;
  }
  // The estimated times of the two, in clocks, fitted to slower forms of both (its K loop and end, the row-tiled kernel's outputs).  Over 123 layers of 50 to
  // 250000 output pixels (3x3 and 1x1, strides one and two) what was picked took 0.2 % longer there than the better of the two in the mean and 8 % at most; with the
  // present kernels, over 109 layers of 64 to 16000 pixels and 64 to 1024 channels, 1.5 % in the mean, 6 % at the 95th percentile, and some few more (512
  // to 192 channels at 6x6, 61 images 21.1, on the small-tile kernel 14.3).  Small-tile kernel / other in those forms, us:
  // 512 channels at 7x7, one image 8.9 / 18.9, eight 13.6 / 19.8; 64 at 56x56, one 5.7 / 8.5, four 9.8 / 9.0, eight 15.2 /
  // 10.0; int8 256 at 14x14, eight 8.3 / 10.9.  Strided 1x1 layers, where the other is the large-tile kernel: 256 to 448 at
  // 20x20, 193 images 34 / 188.  Fully connected, 448 to 3968, 49 images 5.4 / 17.8, 2816 to 3776, 378 images 40 / 30.
  // 1x1, 128 to 128 at 28x28, 64 images 18.6 / 11.0; int8 64 to 128 at 56x56 stride 2, 32 images 16.1 / 10.6.
  double other;
  if (h->point_ok) {
    other = c->rows.cost;                                 // (the large-tile kernel is taken above where it is faster than that)
  } else if (c->kernel == kRows) {
    other = 3900.0 + 1.45 * std::min(c->rows.cost, 22000.0) + 1.05 * std::max(c->rows.cost - 22000.0, 0.0);
  } else {
    const cg::TilePlan& t = c->tile;
    const int rounds = (t.wgs + cg::cu_count() - 1) / cg::cu_count();
    other = 7200.0 + rounds * (7900.0 + (t.stages[0] + 0.29 * t.stages[1]) * (1200.0 + 2.3 * t.cps * t.fp * t.bn));
  }
  if (c->direct.est < other) c->kernel = kDirect;
}

// Two fragments per wavefront write an output twice and read the residual after the first time: where the two may be the
// same memory, a plan with one fragment is kept beside.
void plan_over(const cg_conv* h, CallPlan* c) {
  if (c->kernel != kRows || c->rows.pf != 2 || !(h->d.epilogue & CG_EPI_RESIDUAL)) return;
  cg_conv_desc dn = h->d;
  dn.n_max = c->n;
  c->rows_over = cg::rows_plan(dn, cg::cu_count(), c->rows.cps, 1);
}

// The launch shape follows the batch of the call: a smaller batch than n_max is planned afresh and the
// new plan is used if it reads the prepacked weights the same way.
CallPlan plan_call(const cg_conv* h, int n) {
  CallPlan c = h->first;
  c.n = n;
  cg_conv_desc dn = h->d;
  dn.n_max = n;
  if (h->variant == CG_VARIANT_MFMA_ROWS || h->point_ok) {
    const cg::RowsPlan q = h->point_ok ? cg::point_plan(dn, cg::cu_count()) : cg::rows_plan(dn, cg::cu_count(), c.rows.cps, 2);
    if (q.ok && q.grp_mode == c.rows.grp_mode && q.gsp == c.rows.gsp &&
        q.stages[0] == c.rows.stages[0] && q.stages[1] == c.rows.stages[1])
      c.rows = q;
  }
  if (h->tile_too || (h->variant == CG_VARIANT_TILE && !h->point_ok)) {
    const cg::TilePlan q = cg::tile_plan(dn, cg::cu_count());
    if (q.ok && q.taps == c.tile.taps && q.cps == c.tile.cps && q.wn == c.tile.wn && q.grp_mode == c.tile.grp_mode &&
        q.gsp == c.tile.gsp && q.stages[0] == c.tile.stages[0] && q.stages[1] == c.tile.stages[1])
      c.tile = q;
    else if (h->tile_too)
      c.tile.ok = 0;
  }
  plan_direct(h, n, &c);
  pick_kernel(h, &c);
  plan_over(h, &c);
  return c;
}

CallPlan call_plan(const cg_conv* h, int n) {
  if (n == h->first.n) return h->first;
  std::lock_guard<std::mutex> g(h->lock);
  for (int i = 0; i < cg_conv::kKept; ++i)
    if (h->kept_n[i] == n) return h->kept[i];
  const int at = h->kept_next;
  h->kept_next = (at + 1) % cg_conv::kKept;
  const CallPlan c = plan_call(h, n);
  if (at < (int)h->kept.size())
    h->kept[at] = c;
  else
    h->kept.push_back(c);
  h->kept_n[at] = n;
  return c;
}

// Whether the requantisation of channel c fits 32 bits once its sum is clamped to [lo, hi] (sums beyond give the value that
// the last one gives): every factor below 2^23, every sum below 2^31.  t = S*mult_d + addend + residual*res_mult lies beyond the
// bytes' range on either side at the bounds, whichever mult is taken and whatever the residual is.
bool fits_32_bits(const cg_conv_desc& d, int c, int32_t* addend, int32_t* lo, int32_t* hi) {
  const long long m0 = d.rq_mult0 ? d.rq_mult0[c] : 1, m1 = d.rq_mult1 ? d.rq_mult1[c] : 1, limit = 1ll << 23;
  const long long least = m0 < m1 ? m0 : m1, most = m0 < m1 ? m1 : m0;
  const long long a = (long long)(d.rq_bias ? d.rq_bias[c] : 0) * (1ll << d.rq_shift) + (d.rq_shift > 0 ? 1ll << (d.rq_shift - 1) : 0ll);
  const long long res = (d.epilogue & CG_EPI_RESIDUAL) ? 128ll * (d.rq_res_mult < 0 ? -(long long)d.rq_res_mult : d.rq_res_mult) : 0;
  const long long range = 128ll << d.rq_shift, span = range + (a < 0 ? -a : a) + res;
  if (least <= 0 || most >= limit || res >= 128 * limit || span >= (1ll << 31)) return false;
  const long long bound = span / least + 1;                // at +-bound: |S * mult| > span for either mult
  if (bound >= limit || bound * most + (a < 0 ? -a : a) + res >= (1ll << 31)) return false;
  *addend = (int32_t)a;
  *lo = (int32_t)-bound;
  *hi = (int32_t)bound;
  return true;
}

cg::Params base_params(const cg_conv* h) {
  const cg_conv_desc& d = h->d;
  const char* pk = (const char*)d.packed;
  const Layout& l = h->lay;
  cg::Params p{};
  p.h = d.h;
  p.w = d.w;
  p.c_in = d.c_in;
  p.c_out = d.c_out;
  p.c_base = d.c_base;
  p.c_cond = h->c_cond;
  p.kh = d.kh;
  p.kw = d.kw;
  p.stride = d.stride;
  p.pad = d.pad;
  p.ho = h->ho;
  p.wo = h->wo;
  p.x_pixel_stride = d.x_pixel_stride;
  p.epilogue = d.epilogue;
  p.in_dtype = d.in_dtype;
  p.out_dtype = d.out_dtype;
  p.gated = h->c_cond > 0;
  p.two_sided = d.delta_hi != nullptr;
  p.rq_shift = d.rq_shift;
  p.rq_res_mult = d.rq_res_mult;
  p.words = (d.c_out + 31) / 32;
  p.groups = d.groups > 1 ? d.groups : 1;
  p.cpg = d.c_out / p.groups;
  p.shuffle = d.shuffle;
  const size_t ts = l.table_stride;
  p.thr_f = (const float*)(pk + 0 * ts);
  p.thr_hi_f = (const float*)(pk + 1 * ts);
  p.thr_i = (const int32_t*)(pk + 0 * ts);
  p.sc0 = (const float*)(pk + 2 * ts);
  p.sh0 = (const float*)(pk + 3 * ts);
  p.sc1 = (const float*)(pk + 4 * ts);
  p.sh1 = (const float*)(pk + 5 * ts);
  p.mult0 = (const int32_t*)(pk + 2 * ts);
  p.mult1 = (const int32_t*)(pk + 3 * ts);
  p.bias = (const int32_t*)(pk + 4 * ts);
  p.w_base = pk + l.w_base_off;
  p.w_cond = pk + l.w_cond_off;
  p.table_stride = ts;
  p.zeros = pk + 7 * ts;       // the last table is never written: zeros
  return p;
}

inline uint32_t f2u(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  return u;
}

}  // namespace

namespace {

// Scratch for cg_conv_forward_noalloc: what cg_conv_forward takes as its `workspace` argument (the
// batch's decision bitmap when only counts are asked for, and the first-pass counts and the channel
// mask of the channel-wise gate).  Every GPU the library runs on holds its own copy of the array
// until the process ends.  In host code the array's name is not a device address: the address is
// asked for once per device and kept.
constexpr size_t kScratchBytes = (size_t)16 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
void* g_scratch_ptr[kMaxDevices] = {};

// the current device's copy of `scratch` (NULL with the error text set on failure)
void* scratch_of_current_device() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    fail(CG_EHIP, "no usable current device for the scratch array: %s", hipGetErrorString(e));
    return nullptr;
  }
  void* ptr = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
  if (ptr) return ptr;
  e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    fail(CG_EHIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
    return nullptr;
  }
  __atomic_store_n(&g_scratch_ptr[dev], ptr, __ATOMIC_RELEASE);   // (two threads may both ask: same answer)
  return ptr;
}

// A word of pinned host memory that any GPU's kernels can write, held until the process ends: a kernel whose bounded wait
// came to its end sets it (a mistake in this library: the pass's results are wrong).  NULL with the error text set on failure.
std::mutex g_gave_up_lock;
uint32_t* g_gave_up = nullptr;

uint32_t* gave_up_word() {
  std::lock_guard<std::mutex> g(g_gave_up_lock);
  if (g_gave_up) return g_gave_up;
  void* ptr = nullptr;
  const hipError_t e = hipHostMalloc(&ptr, 64, hipHostMallocPortable | hipHostMallocMapped);
  if (e != hipSuccess || !ptr) {
    fail(CG_EHIP, "hipHostMalloc of the kernels' error word failed: %s", hipGetErrorString(e));
    return nullptr;
  }
  memset(ptr, 0, 64);
  return g_gave_up = (uint32_t*)ptr;
}

}  // namespace

extern "C" {

const char* cg_last_error(void) { return g_err.c_str(); }

size_t cg_conv_packed_bytes(const cg_conv_desc* desc) {
  int ho, wo;
  if (validate(desc, &ho, &wo) != CG_OK) return 0;
  Plans pl;
  if (resolve_variant(*desc, &pl) != CG_OK) return 0;
  return make_layout(*desc, pl.wpk_base_bytes, pl.wpk_cond_bytes, pl.wpd_base_bytes, pl.wpd_cond_bytes, pl.wpt_base_bytes).total;
}

int cg_conv_create(cg_conv** out, const cg_conv_desc* desc, void* hip_stream) {
  if (!out) return fail(CG_EINVAL, "out is NULL");
  *out = nullptr;
  int ho, wo;
  int rc = validate(desc, &ho, &wo);
  if (rc != CG_OK) return rc;
  const cg_conv_desc& d = *desc;
  Plans pl;
  rc = resolve_variant(d, &pl);
  if (rc != CG_OK) return rc;
  const int variant = pl.variant;
  const Layout lay = make_layout(d, pl.wpk_base_bytes, pl.wpk_cond_bytes, pl.wpd_base_bytes, pl.wpd_cond_bytes, pl.wpt_base_bytes);
  if (!d.packed) return fail(CG_EINVAL, "packed is NULL");
  if (((uintptr_t)d.packed & 255) != 0) return fail(CG_EINVAL, "packed must be 256-byte aligned");
  if (d.packed_bytes < lay.total)
    return fail(CG_EINVAL, "packed_bytes %zu is smaller than the %zu required", d.packed_bytes, lay.total);

  cg_conv* h = new (std::nothrow) cg_conv();
  if (!h) return fail(CG_ENOMEM, "out of host memory");
  h->d = d;
  if (h->d.x_pixel_stride == 0) h->d.x_pixel_stride = d.c_in;
  h->ho = ho;
  h->wo = wo;
  h->c_cond = d.c_in - d.c_base;
  h->variant = variant;
  h->direct_ok = pl.direct_ok;
  h->point_ok = pl.point_ok;
  h->tile_too = pl.tile_too;
  h->lay = lay;
  h->first.n = d.n_max;
  h->first.rows = pl.v3;
  h->first.tile = pl.v4;
  plan_direct(h, d.n_max, &h->first);
  pick_kernel(h, &h->first);
  plan_over(h, &h->first);
  h->base = base_params(h);

  // Host image of the per-channel tables.
  //   float path: 0 thr, 1 thr_hi, 2 sc0, 3 sh0, 4 sc1, 5 sh1
  //   int path:   0 thr, 2 mult0, 3 mult1, 4 bias; 5 and 6, of every 64 channels: (bias << shift) + half as 64-bit
  //               words, 32 channels in table 5 and 32 in table 6; where 32 bits are enough (fits_32_bits, all channels):
  //               1 and 6 the bounds of the sum, 5 the same addend in 32 bits
  const size_t tw = lay.table_stride / 4;
  try {
    h->staging.assign(tw * kTables, 0u);
    h->kept.reserve(cg_conv::kKept);
  } catch (...) {
    delete h;
    return fail(CG_ENOMEM, "out of host memory");
  }
  uint32_t* t = h->staging.data();
  const bool gated = d.c_base < d.c_in;
  const float inf = std::numeric_limits<float>::infinity();
  int32_t fit_add, fit_lo, fit_hi;
  bool fits = d.in_dtype == CG_I8 && d.out_dtype == CG_I8;
  for (int c = 0; fits && c < d.c_out; ++c) fits = fits_32_bits(d, c, &fit_add, &fit_lo, &fit_hi);
  h->base.fit32 = fits;
  for (int c = 0; c < d.c_out; ++c) {
    if (d.in_dtype == CG_I8) {
      t[0 * tw + c] = (uint32_t)(gated ? d.gate_thr_i32[c] : std::numeric_limits<int32_t>::min());
      t[2 * tw + c] = (uint32_t)(d.rq_mult0 ? d.rq_mult0[c] : 1);
      t[3 * tw + c] = (uint32_t)(d.rq_mult1 ? d.rq_mult1[c] : 1);
      t[4 * tw + c] = (uint32_t)(d.rq_bias ? d.rq_bias[c] : 0);
      const uint64_t add = (uint64_t)((long long)(d.rq_bias ? d.rq_bias[c] : 0) * (1ll << d.rq_shift) +
                                      (d.rq_shift > 0 ? 1ll << (d.rq_shift - 1) : 0ll));
      if (fits && fits_32_bits(d, c, &fit_add, &fit_lo, &fit_hi)) {
        t[1 * tw + c] = (uint32_t)fit_lo;
        t[5 * tw + c] = (uint32_t)fit_add;
        t[6 * tw + c] = (uint32_t)fit_hi;
        continue;
      }
      uint32_t* pair = t + (5 + c % 64 / 32) * tw + c / 64 * 64 + 2 * (c % 32);
      pair[0] = (uint32_t)add;
      pair[1] = (uint32_t)(add >> 32);
    } else {
      float lo = -inf, hi = inf;
      if (gated) {
        // merged gate: compare the raw partial sum with E + Delta*sqrt(Var+eps); never form inf*0
        const double sd = std::sqrt((double)d.gate_var[c] + (double)d.gate_eps);
        const double dl = d.delta[c];
        lo = std::isinf(dl) ? (dl < 0 ? -inf : inf) : (float)((double)d.gate_mean[c] + dl * sd);
        if (d.delta_hi) {
          const double dh = d.delta_hi[c];
          hi = std::isinf(dh) ? (dh < 0 ? -inf : inf) : (float)((double)d.gate_mean[c] + dh * sd);
        }
      }
      t[0 * tw + c] = f2u(lo);
      t[1 * tw + c] = f2u(hi);
      t[2 * tw + c] = f2u(d.scale0 ? d.scale0[c] : 1.0f);
      t[3 * tw + c] = f2u(d.shift0 ? d.shift0[c] : 0.0f);
      t[4 * tw + c] = f2u(d.scale1 ? d.scale1[c] : 1.0f);
      t[5 * tw + c] = f2u(d.shift1 ? d.shift1[c] : 0.0f);
    }
  }
  h->base.one_pair = d.in_dtype != CG_I8 && memcmp(t + 2 * tw, t + 4 * tw, (size_t)d.c_out * 4) == 0 &&
                     memcmp(t + 3 * tw, t + 5 * tw, (size_t)d.c_out * 4) == 0;
  // host pointers must not be used after create
  h->d.gate_mean = h->d.gate_var = h->d.delta = h->d.delta_hi = nullptr;
  h->d.gate_thr_i32 = nullptr;
  h->d.scale0 = h->d.shift0 = h->d.scale1 = h->d.shift1 = nullptr;
  h->d.rq_mult0 = h->d.rq_mult1 = h->d.rq_bias = nullptr;

  hipStream_t s = (hipStream_t)hip_stream;
  char* pk = (char*)d.packed;
  hipError_t e = hipMemcpyAsync(pk, t, lay.table_stride * kTables, hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(pk + lay.w_base_off, d.w_base, lay.w_base_bytes, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && lay.w_cond_bytes)
    e = hipMemcpyAsync(pk + lay.w_cond_off, d.w_cond, lay.w_cond_bytes, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && variant == CG_VARIANT_TILE && !pl.point_ok)
    e = cg::launch_tile_pack(pl.v4, h->base, pk + lay.wpk_base_off, pk + lay.wpk_cond_off, s);
  if (e == hipSuccess && (variant == CG_VARIANT_MFMA_ROWS || pl.point_ok))
    e = cg::launch_rows_pack(pl.v3, h->base, pk + lay.wpk_base_off, pk + lay.wpk_cond_off, s);
  if (e == hipSuccess && pl.tile_too)
    e = cg::launch_tile_pack(pl.v4, h->base, pk + lay.wpt_base_off, nullptr, s);
  if (e == hipSuccess && pl.direct_ok)
    e = cg::launch_direct_pack(pl.vd, h->base, pk + lay.wpd_base_off, pk + lay.wpd_cond_off, s);
  if (e != hipSuccess) {
    const int code = fail(CG_EHIP, "cg_conv_create: %s", hipGetErrorString(e));
    delete h;
    return code;
  }
  h->d.w_base = h->d.w_cond = nullptr;
  // set-up is the place to ask for this device's scratch address and the kernels' error word, so that a later
  // forward call (possibly under graph capture) only reads them
  h->base.gave_up = gave_up_word();
  if (!h->base.gave_up || !scratch_of_current_device()) {
    const std::string keep = g_err;
    delete h;
    g_err = keep;
    return CG_EHIP;
  }
  *out = h;
  return CG_OK;
}

namespace {
// Workspace layout: [decisions: the batch's bitmap, or (kCounting) its counts][channel mask].  Fired gates
// are counted from a decision bitmap; it goes to the workspace when the caller asks for counts without a bitmap, and so
// does the first pass of the channel-wise gate.  The mask exists only with the channel-wise gate.
struct WsLayout {
  size_t dec_off, dec_bytes, mask_off, mask_bytes, total;
};
// What a call gets of it: what any call may need (the caller's workspace); what this call needs; or what the plain kernel
// needs when it counts the fired gates itself (an image whose bitmap does not fit the scratch array).
enum Scratch { kAnyCall, kThisCall, kCounting };
WsLayout ws_layout(const cg_conv* h, int32_t n, Scratch mode, bool counts_only) {
  WsLayout w{};
  const size_t words = (size_t)(h->d.c_out + 31) / 32;
  const bool gated = h->c_cond > 0, chan_gate = gated && h->d.tau_c > 0.0f;
  if (mode == kCounting)
    w.dec_bytes = chan_gate ? align256((size_t)n * h->d.c_out * 4 + 8) : 0;
  else if (gated && (mode == kAnyCall || chan_gate || counts_only))
    w.dec_bytes = align256((size_t)n * h->ho * h->wo * words * 4);
  if (chan_gate) w.mask_bytes = align256((size_t)n * words * 4);
  w.dec_off = 0;
  w.mask_off = w.dec_bytes;
  w.total = w.mask_off + w.mask_bytes;
  return w;
}
}  // namespace

size_t cg_conv_workspace_bytes(const cg_conv* h, int32_t n) {
  if (!h || n <= 0) return 0;
  return ws_layout(h, n, kAnyCall, true).total;
}

int cg_conv_info(const cg_conv* h, int32_t* ho, int32_t* wo) {
  if (!h) return -1;
  if (ho) *ho = h->ho;
  if (wo) *wo = h->wo;
  return h->variant;
}

}  // extern "C"

namespace {

// counts: [n][c_out] fired counts; total: their sum, cleared first if clear_total (both NULL or neither)
int forward_impl(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap,
                 uint32_t* counts, uint32_t* total, bool clear_total, Scratch mode, void* workspace, size_t workspace_bytes,
                 void* hip_stream, cg::Beside* beside = nullptr);

}  // namespace

extern "C" {

int cg_conv_forward(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap,
                    uint32_t* counts, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return forward_impl(h, n, x, residual, y, bitmap, counts ? counts + 2 : nullptr, counts, true, kAnyCall, workspace,
                      workspace_bytes, hip_stream);
}

size_t cg_conv_call_scratch_bytes(const cg_conv* h, int32_t n, int has_bitmap, int has_counts) {
  if (!h || n <= 0) return 0;
  return ws_layout(h, n, kThisCall, has_counts && !has_bitmap).total;
}

int cg_conv_call(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap, uint32_t* counts, void* workspace,
                 size_t workspace_bytes, void* hip_stream) {
  return forward_impl(h, n, x, residual, y, bitmap, counts ? counts + 2 : nullptr, counts, true, kThisCall, workspace, workspace_bytes, hip_stream);
}

int cg_conv_call_beside(cg_conv* h, int32_t n, const void* x, void* y, const void* w1, const float* scale1, const float* shift1, void* y1, int32_t c_out1,
                        int32_t relu1, void* hip_stream) {
  if (!h) return fail(CG_EINVAL, "handle is NULL");
  const cg_conv_desc& d = h->d;
  if (d.in_dtype != CG_BF16 || d.x_pixel_stride != d.c_in) return fail(CG_EUNSUPPORTED, "cg_conv_call_beside: bf16 layers of whole pixels only");
  if (d.epilogue & CG_EPI_RESIDUAL) return fail(CG_EUNSUPPORTED, "cg_conv_call_beside: layers without a residual only");
  if (d.tau_c > 0.0f) return fail(CG_EUNSUPPORTED, "cg_conv_call_beside: no channel-wise gate");
  if (h->ho != (d.h - 1) / d.stride + 1 || h->wo != (d.w - 1) / d.stride + 1)
    return fail(CG_EUNSUPPORTED, "cg_conv_call_beside: layers whose output has the size of the 1x1's only");
  const int rc = cg::point_check(x, w1, scale1, shift1, y1, n, d.h, d.w, d.c_in, c_out1, d.stride);
  if (rc != CG_OK || n == 0) return rc;
  // One launch where the layer runs on the small-tile kernel with its K split and the 1x1 would run in small pieces, else two.
  cg::Beside both{cg::point_args(x, w1, scale1, shift1, y1, n, d.h, d.w, d.c_in, c_out1, d.stride, relu1), false};
  const bool pieces = cg::point_in_pieces((long long)n * both.what.ho * both.what.wo, c_out1, cg::cu_count());
  const int first = forward_impl(h, n, x, nullptr, y, nullptr, nullptr, nullptr, true, kThisCall, nullptr, 0, hip_stream, pieces ? &both : nullptr);
  if (first != CG_OK || both.done) return first;
  return cg_pointwise_conv(x, w1, scale1, shift1, y1, n, d.h, d.w, d.c_in, c_out1, d.stride, relu1, hip_stream);
}

int cg_conv_forward_noalloc(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap,
                            uint32_t* counts, void* hip_stream) {
  if (!h) return fail(CG_EINVAL, "handle is NULL");
  if (n < 0 || n > h->d.n_max) return fail(CG_EINVAL, "n = %d is outside [0, n_max = %d]", n, h->d.n_max);
  if (n == 0) return CG_OK;
  Scratch mode = kAnyCall;
  int step = n;                          // images at a time
  if (h->variant == CG_VARIANT_NAIVE) {
    // Layers of this family take any batch: as many images at a time as the scratch array serves, and one at a time,
    // counted without a bitmap, where not even one image's bitmap fits.
    const bool counts_only = counts && !bitmap;
    mode = kThisCall;
    if (ws_layout(h, n, mode, counts_only).total > kScratchBytes) {
      const size_t one = ws_layout(h, 1, mode, counts_only).total;
      if (one > kScratchBytes) mode = kCounting;
      step = one > kScratchBytes ? 1 : (int)(kScratchBytes / one);
    }
  }
  const size_t need = mode == kAnyCall ? cg_conv_workspace_bytes(h, n) : 0;
  if (need > kScratchBytes)
    return fail(CG_EUNSUPPORTED, "this call needs %zu bytes of scratch; the library's fixed scratch array holds %zu",
                need, kScratchBytes);
  void* ws = scratch_of_current_device();
  if (!ws) return CG_EHIP;
  if (step == n)
    return forward_impl(h, n, x, residual, y, bitmap, counts ? counts + 2 : nullptr, counts, true, mode, ws, kScratchBytes,
                        hip_stream);
  if (!x || !y) return fail(CG_EINVAL, "x and y must not be NULL");
  const cg_conv_desc& d = h->d;
  const size_t xi = (size_t)d.h * d.w * d.x_pixel_stride * elem_bytes(d.in_dtype), px = (size_t)h->ho * h->wo;
  const size_t yi = px * d.c_out * elem_bytes(d.out_dtype);
  const size_t ri = px * d.c_out * elem_bytes(d.in_dtype == CG_I8 ? CG_I8 : d.out_dtype);
  for (int i = 0; i < n; i += step) {
    const int m = n - i < step ? n - i : step;
    const int rc = forward_impl(h, m, (const char*)x + i * xi, residual ? (const char*)residual + i * ri : nullptr,
                                (char*)y + i * yi, bitmap ? bitmap + i * px * ((d.c_out + 31) / 32) : nullptr,
                                counts ? counts + 2 + (size_t)i * d.c_out : nullptr, counts, i == 0, mode, ws, kScratchBytes,
                                hip_stream);
    if (rc != CG_OK) return rc;
  }
  return CG_OK;
}

void cg_conv_destroy(cg_conv* h) { delete h; }

}  // extern "C"

namespace {

int forward_impl(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap,
                 uint32_t* counts, uint32_t* total, bool clear_total, Scratch mode, void* workspace, size_t workspace_bytes,
                 void* hip_stream, cg::Beside* beside) {
  if (!h) return fail(CG_EINVAL, "handle is NULL");
  if (n < 0 || n > h->d.n_max) return fail(CG_EINVAL, "n = %d is outside [0, n_max = %d]", n, h->d.n_max);
  if (n == 0) return CG_OK;
  if (__atomic_load_n(h->base.gave_up, __ATOMIC_RELAXED))
    return fail(CG_EHIP, "a kernel of an earlier call gave up waiting for its own loads; that call's results are wrong");
  if (!x || !y) return fail(CG_EINVAL, "x and y must not be NULL");
  if ((h->d.epilogue & CG_EPI_RESIDUAL) && !residual)
    return fail(CG_EINVAL, "residual is NULL but the layer was created with CG_EPI_RESIDUAL");
  if (total && ((uintptr_t)total & 7)) return fail(CG_EINVAL, "counts must be 8-byte aligned");
  const bool aligned = ((((uintptr_t)x) | ((uintptr_t)y) | ((uintptr_t)residual) | ((uintptr_t)bitmap)) & 15) == 0;
  if (h->variant != CG_VARIANT_NAIVE && !aligned)
    return fail(CG_EINVAL, "x, y, residual and bitmap must be 16-byte aligned");
  CallPlan cp = call_plan(h, n);
  const WsLayout wl = ws_layout(h, n, mode, counts && !bitmap);
  const size_t need = wl.total;
  if (need > 0 && (!workspace || workspace_bytes < need))
    return fail(CG_EINVAL, "workspace of %zu bytes is smaller than the %zu required", workspace_bytes, need);
  if (need > 0 && ((uintptr_t)workspace & 255)) return fail(CG_EINVAL, "workspace must be 256-byte aligned");

  const cg_conv_desc& d = h->d;
  const char* pk = (const char*)d.packed;
  const Layout& l = h->lay;
  cg::Params p = h->base;
  p.n = n;
  p.m_total = (long long)n * h->ho * h->wo;
  p.x = x;
  p.residual = residual;
  p.y = y;
  p.bitmap = bitmap;
  p.counts = counts;
  p.total = total;
  p.clear_total = counts && clear_total;

  if (!aligned || mode == kCounting) cp.kernel = kNaive;      // (the plain kernel is the layer's family: the others were turned away)
  if (cp.kernel == kRows && cp.rows.pf == 2 && residual) {
    // (see plan_over)
    const char *y0 = (const char*)y, *r0 = (const char*)residual;
    const size_t len = (size_t)p.m_total * d.c_out * 2;
    if (y0 < r0 + len && r0 < y0 + len) cp.rows = cp.rows_over;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  char* ws = (char*)workspace;
  auto launch = [&](const cg::Params& q) -> hipError_t {
    switch (cp.kernel) {
      case kRows: return cg::launch_rows(cp.rows, q, pk + l.wpk_base_off, pk + l.wpk_cond_off, s);
      case kTile: return cg::launch_tile(cp.tile, q, pk + (h->tile_too ? l.wpt_base_off : l.wpk_base_off), pk + l.wpk_cond_off, s);
      case kDirect: {
        hipError_t err = hipSuccess;
        for (int i = 0; i < n && err == hipSuccess; i += cp.piece) {
          const long long px = (long long)h->ho * h->wo, oi = i * px * d.c_out;
          cg::Params r = q;
          r.n = n - i < cp.piece ? n - i : cp.piece;
          r.m_total = r.n * px;
          r.x = (const char*)q.x + (long long)i * d.h * d.w * d.x_pixel_stride * elem_bytes(d.in_dtype);
          r.residual = (const char*)q.residual + (q.residual ? oi * elem_bytes(d.in_dtype == CG_I8 ? CG_I8 : d.out_dtype) : 0);
          r.y = (char*)q.y + (q.y ? oi * elem_bytes(d.out_dtype) : 0);
          if (q.bitmap) r.bitmap = q.bitmap + i * px * q.words;
          if (q.chan_mask) r.chan_mask = q.chan_mask + (long long)i * q.words;
          r.clear_total = q.clear_total && i == 0;
          // (a batch in one piece, and the layer's only pass)
          const bool both = beside && cp.piece >= n && d.tau_c <= 0.0f && cg::takes_beside(cp.direct, r);
          err = cg::launch_direct(r.n == cp.piece ? cp.direct : cp.direct_rest, r, pk + l.wpd_base_off, pk + l.wpd_cond_off, s, both ? &beside->what : nullptr);
          if (both) beside->done = true;
        }
        return err;
      }
      default: return cg::launch_naive(q, s);
    }
  };
  hipError_t e = hipSuccess;
  if (p.gated && d.tau_c > 0.0f) {
    // Channel-wise gate (Sec. 3.2): a first pass over the base path and the gate gives the decisions,
    // counted per (image, channel); the channels at or above tau_c * Ho * Wo form the mask that the
    // full pass ANDs into its decisions.
    const double need_d = std::ceil((double)d.tau_c * (double)((long long)h->ho * h->wo));
    const uint32_t need_u = need_d >= 4294967295.0 ? 0xffffffffu : (uint32_t)need_d;
    uint32_t* mask = (uint32_t*)(ws + wl.mask_off);
    cg::Params q = p;
    q.gate_only = 1;
    q.y = nullptr;
    q.counts = q.total = nullptr;
    q.clear_total = 0;
    q.bitmap = nullptr;
    if (mode == kCounting) {
      q.total = (uint32_t*)(ws + wl.dec_off);
      q.counts = q.total + 2;
      q.count_here = 1;
      e = cg::launch_zero_u32(q.total, 2 + (size_t)n * d.c_out, s);
      if (e == hipSuccess) e = launch(q);
      if (e == hipSuccess) e = cg::launch_counts_chan_mask(q, q.counts, need_u, mask, s);
    } else {
      q.bitmap = (uint32_t*)(ws + wl.dec_off);
      e = launch(q);
      if (e == hipSuccess) e = cg::launch_bitmap_chan_mask(q, q.bitmap, need_u, mask, s);
    }
    p.chan_mask = mask;
  }
  if (e == hipSuccess && counts && (!p.gated || mode == kCounting))       // (the first call's counts follow the total)
    e = clear_total ? cg::launch_zero_u32(total, 2 + (size_t)n * d.c_out, s) : cg::launch_zero_u32(counts, (size_t)n * d.c_out, s);
  if (!p.gated) {
    // a dense layer has no decisions
    if (e == hipSuccess && bitmap) e = cg::launch_zero_u32(bitmap, (size_t)p.m_total * p.words, s);
    p.counts = p.total = nullptr;
    p.clear_total = 0;
    p.bitmap = nullptr;
  } else if (counts && mode == kCounting) {
    p.count_here = 1;
    p.clear_total = 0;
  } else if (counts && !bitmap) {
    p.bitmap = (uint32_t*)(ws + wl.dec_off);      // free again once the mask exists
  }
  if (e == hipSuccess) e = launch(p);
  if (e == hipSuccess && counts && p.gated && !p.count_here) e = cg::launch_bitmap_counts(p, p.bitmap, s);
  if (e != hipSuccess) return fail(CG_EHIP, "cg_conv_forward: %s", hipGetErrorString(e));
  return CG_OK;
}

}  // namespace
