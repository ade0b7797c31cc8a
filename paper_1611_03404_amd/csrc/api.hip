// Host side of libceleste: the C ABI, argument validation, packing of ragged
// batches into device metadata (sources -> images -> work items), and the
// drivers of the evaluation and of the trust-region fits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "celeste_internal.h"
#include "host_team.h"

using namespace celeste;

namespace celeste {
hipError_t launch_fit_start(FitDev st, int n_src, hipStream_t s);
}

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

}  // namespace

namespace celeste {
void set_error(const char* msg) { g_err = msg; }
}  // namespace celeste

namespace {

#define HIPCHK(x)                                                                          \
  do {                                                                                     \
    hipError_t e_ = (x);                                                                   \
    if (e_ != hipSuccess) return fail(CELESTE_E_DEVICE, "%s: %s", #x, hipGetErrorString(e_)); \
  } while (0)

#define CHK(x)                 \
  do {                         \
    int r_ = (x);              \
    if (r_ != CELESTE_OK) return r_; \
  } while (0)

struct DevBuf {
  void* p = nullptr;
  size_t cap = 0;
};

}  // namespace

struct celeste_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  int chunk_px = 4096;
  int block = 256;
  int use_graph = 1;
  int variant = 3;   // pixel-kernel variant (register budget / unrolling), see CELESTE_OPT_VARIANT
  int tile_log2 = 3;     // log2 tile width of the value+gradient+Hessian kernel
  float e_zero = -160.f; // exact-zero threshold of the pixel kernels (log2 density)
  bool exp2_flushes = false;   // the device's exp2 returns 0 below 2^-126 (checked at creation)
  int vblock = 256;      // value kernel block size
  int vtile_log2 = 3;    // log2 tile width of the value kernel
  DevBuf meta, items_kept;                // packed metadata (one upload); a subsample's work items and kept rows
  DevBuf imgs, items, srcs;               // where the last pack's parts lie in them (views, not owned)
  DevBuf tables, partials, img_const, staging, theta, o_elbo;
  DevBuf st_buf;   // all trust-region state in one allocation
  DevBuf ctr;      // device counters: pixel evaluations [full, value, grad], subproblem paths and work [3..8]
  int profile = 0;
  celeste_stats stats{};

  celeste_net* net = nullptr;   // surrogate network (not owned)
  DevBuf sur;                   // surrogate predictions (float, S x 27)
  DevBuf tile_off, img_field, nbr_off;             // crowded-field index buffers
  DevBuf tables2, fsky, theta_flag;                // second setup table (field updates), field skies, estimates' check
  DevBuf lr_in, lr_cov, lr_status, lr_eval;        // linear-response covariance staging
  DevBuf lfact;                                    // log n! table of the pixel constants
  DevBuf lb_buf;                                   // L-BFGS state beyond the fit state
  DevBuf imgs_s, items_s, srcs_s, partials_s;      // the pixel-subsampled pack of a fit's early phase
  int persistent = -1;                             // fits: persistent pixel-kernel blocks per CU (0: off,
                                                   // -1: as many as the kernel instance keeps resident)
  int pgrid = 0;                                   // the current fit's persistent grid (blocks)
  int tr_chol = 1;                                 // fits: subproblem by Cholesky where -H is positive definite
  int fp64_sums = 0;                               // value+gradient+Hessian kernel: FP64 sums per tile step
  int trial_derivs = 1;                            // fits: gradient and Hessian evaluated at the trial point
  int n_cu = 0;                                    // compute units of the device
  DevBuf qbuf;                                     // the fits' device work queue
  bool lfact_ready = false;
  DevBuf h_meta, h_items, h_lists;                 // pinned host staging: packed metadata, a subsample's items,
                                                   // tile lists,
  DevBuf h_poll, h_flags;                          // active counts of a fit's last two polls; theta_flag read back
  DevBuf h_ring;                                   // pixels and results of host batches on their way: two pieces
  hipEvent_t ring_ev[2] = {};                      // a piece's last copy, and whether there was one
  bool ring_used[2] = {};
  size_t ring_mapped = 0;                          // bytes of it, from its start, that have been used before
};

namespace {
// The value+gradient+Hessian kernel's variant with the context's summation precision (bit 3).
int full_variant(const celeste_ctx* c) { return c->variant | (c->fp64_sums ? 8 : 0); }
}  // namespace

namespace celeste {
int ctx_device(const celeste_ctx* c) { return c->device; }
hipStream_t ctx_stream(const celeste_ctx* c) { return c->stream; }
}  // namespace celeste

namespace {

int ensure(DevBuf& b, size_t bytes) {
  if (bytes == 0) bytes = 16;
  if (bytes <= b.cap) return CELESTE_OK;
  if (b.p) (void)hipFree(b.p);
  b.p = nullptr;
  b.cap = 0;
  if (hipMalloc(&b.p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(CELESTE_E_NOMEM, "device allocation of %zu bytes failed", bytes);
  }
  b.cap = bytes;
  return CELESTE_OK;
}

// Pinned host buffer of at least `bytes` (contents not kept on growth).
int ensure_host(DevBuf& b, size_t bytes) {
  if (bytes == 0) bytes = 16;
  if (bytes <= b.cap) return CELESTE_OK;
  const size_t cap = std::max(bytes, b.cap + b.cap / 2);
  if (b.p) (void)hipHostFree(b.p);
  b.p = nullptr;
  b.cap = 0;
  if (hipHostMalloc(&b.p, cap, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    b.p = nullptr;
    return fail(CELESTE_E_NOMEM, "pinned host allocation of %zu bytes failed", cap);
  }
  b.cap = cap;
  return CELESTE_OK;
}

template <class T>
T* as(DevBuf& b) {
  return static_cast<T*>(b.p);
}

bool finite(double x) { return std::isfinite(x); }

// Cholesky of a symmetric 4x4; false if not positive definite.
bool chol4(const double A[4][4], double L[4][4]) {
  for (int i = 0; i < 4; ++i)
    for (int j = 0; j < 4; ++j) L[i][j] = 0.0;
  for (int j = 0; j < 4; ++j) {
    double d = A[j][j];
    for (int k = 0; k < j; ++k) d -= L[j][k] * L[j][k];
    if (!(d > 0.0)) return false;
    L[j][j] = std::sqrt(d);
    for (int i = j + 1; i < 4; ++i) {
      double v = A[i][j];
      for (int k = 0; k < j; ++k) v -= L[i][k] * L[j][k];
      L[i][j] = v / L[j][j];
    }
  }
  return true;
}

int make_prior(const celeste_prior* p, PriorDev* d) {
  if (!p) return fail(CELESTE_E_INVALID, "prior is NULL");
  if (!(p->p_star > 0.0 && p->p_star < 1.0)) return fail(CELESTE_E_INVALID, "prior p_star must lie in (0,1)");
  std::memset(d, 0, sizeof(*d));
  d->p_star = p->p_star;
  for (int t = 0; t < 2; ++t) {
    if (!finite(p->r_mean[t]) || !(p->r_var[t] > 0.0) || !finite(p->r_var[t]))
      return fail(CELESTE_E_INVALID, "prior r_mean/r_var[%d] invalid", t);
    d->r_mean[t] = p->r_mean[t];
    d->r_var[t] = p->r_var[t];
    for (int j = 0; j < 4; ++j) {
      if (!finite(p->c_mean[t][j])) return fail(CELESTE_E_INVALID, "prior c_mean not finite");
      d->c_mean[t][j] = p->c_mean[t][j];
      d->c_diag[t][j] = p->c_cov[t][j][j];
      for (int k = 0; k < 4; ++k)
        if (!finite(p->c_cov[t][j][k]) || p->c_cov[t][j][k] != p->c_cov[t][k][j])
          return fail(CELESTE_E_INVALID, "prior c_cov[%d] must be finite and symmetric", t);
    }
    double L[4][4];
    if (!chol4(p->c_cov[t], L)) return fail(CELESTE_E_INVALID, "prior c_cov[%d] not positive definite", t);
    double ld = 0.0;
    for (int j = 0; j < 4; ++j) ld += 2.0 * std::log(L[j][j]);
    d->c_logdet[t] = ld;
    // inverse from the Cholesky factor: solve L L^T X = I
    for (int c = 0; c < 4; ++c) {
      double y[4], x[4];
      for (int i = 0; i < 4; ++i) {
        double v = (i == c) ? 1.0 : 0.0;
        for (int k = 0; k < i; ++k) v -= L[i][k] * y[k];
        y[i] = v / L[i][i];
      }
      for (int i = 3; i >= 0; --i) {
        double v = y[i];
        for (int k = i + 1; k < 4; ++k) v -= L[k][i] * x[k];
        x[i] = v / L[i][i];
      }
      for (int i = 0; i < 4; ++i) d->c_inv[t][i][c] = x[i];
    }
  }
  return CELESTE_OK;
}

int make_profiles(const celeste_profiles* p, ProfDev* d) {
  if (!p) return fail(CELESTE_E_INVALID, "profiles is NULL");
  if (p->n_exp < 1 || p->n_exp > CELESTE_MAX_PROTO || p->n_dev < 1 || p->n_dev > CELESTE_MAX_PROTO)
    return fail(CELESTE_E_INVALID, "profile component counts must be in 1..%d", CELESTE_MAX_PROTO);
  std::memset(d, 0, sizeof(*d));
  d->n_exp = p->n_exp;
  d->n_dev = p->n_dev;
  for (int j = 0; j < p->n_exp; ++j) {
    if (!(p->exp_amp[j] >= 0.0) || !finite(p->exp_amp[j]) || !(p->exp_var[j] > 0.0) || !finite(p->exp_var[j]))
      return fail(CELESTE_E_INVALID, "exp profile component %d invalid", j);
    d->amp[j] = p->exp_amp[j];
    d->var[j] = p->exp_var[j];
  }
  for (int j = 0; j < p->n_dev; ++j) {
    if (!(p->dev_amp[j] >= 0.0) || !finite(p->dev_amp[j]) || !(p->dev_var[j] > 0.0) || !finite(p->dev_var[j]))
      return fail(CELESTE_E_INVALID, "dev profile component %d invalid", j);
    d->amp[p->n_exp + j] = p->dev_amp[j];
    d->var[p->n_exp + j] = p->dev_var[j];
  }
  return CELESTE_OK;
}

int check_image(const celeste_image& im, int64_t idx) {
  if (im.band < 0 || im.band > 4) return fail(CELESTE_E_INVALID, "image %lld: band %d not in 0..4", (long long)idx, im.band);
  if (im.h < 1 || im.w < 1 || im.pitch < im.w)
    return fail(CELESTE_E_INVALID, "image %lld: bad shape h=%d w=%d pitch=%d", (long long)idx, im.h, im.w, im.pitch);
  if ((int64_t)im.h * im.w > (int64_t)1 << 30) return fail(CELESTE_E_INVALID, "image %lld: patch too large", (long long)idx);
  if (im.n_psf < 1 || im.n_psf > CELESTE_MAX_PSF)
    return fail(CELESTE_E_INVALID, "image %lld: n_psf %d not in 1..%d", (long long)idx, im.n_psf, CELESTE_MAX_PSF);
  if (im.nbr_pitch != 0 && im.nbr_pitch < im.w)
    return fail(CELESTE_E_INVALID, "image %lld: nbr_pitch must be 0 or >= w", (long long)idx);
  if (!im.pixels) return fail(CELESTE_E_INVALID, "image %lld: pixels is NULL", (long long)idx);
  if (!(im.sky > 0.0) || !finite(im.sky) || !(im.calib > 0.0) || !finite(im.calib))
    return fail(CELESTE_E_INVALID, "image %lld: sky and calib must be positive and finite", (long long)idx);
  for (int k = 0; k < 2; ++k)
    if (!finite(im.origin[k])) return fail(CELESTE_E_INVALID, "image %lld: origin not finite", (long long)idx);
  for (int k = 0; k < 6; ++k)
    if (!finite(im.wcs[k])) return fail(CELESTE_E_INVALID, "image %lld: wcs not finite", (long long)idx);
  if (std::fabs(im.wcs[0] * im.wcs[3] - im.wcs[1] * im.wcs[2]) < 1e-12)
    return fail(CELESTE_E_INVALID, "image %lld: singular WCS matrix", (long long)idx);
  for (int k = 0; k < im.n_psf; ++k) {
    const double* p = im.psf[k];
    for (int j = 0; j < 6; ++j)
      if (!finite(p[j])) return fail(CELESTE_E_INVALID, "image %lld: psf not finite", (long long)idx);
    if (!(p[0] >= 0.0) || !(p[3] > 0.0) || !(p[5] > 0.0) || !(p[3] * p[5] - p[4] * p[4] > 0.0))
      return fail(CELESTE_E_INVALID, "image %lld: psf component %d needs weight >= 0 and a PD covariance",
                  (long long)idx, k);
  }
  return CELESTE_OK;
}

int check_theta(const double* th, int64_t s) {
  for (int i = 0; i < NP; ++i)
    if (!finite(th[i])) return fail(CELESTE_E_INVALID, "theta[%lld][%d] not finite", (long long)s, i);
  if (!(th[2] > 0.0 && th[2] < 1.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: a must lie in (0,1)", (long long)s);
  if (!(th[3] >= 0.0 && th[3] <= 1.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: e_dev must lie in [0,1]", (long long)s);
  if (!(th[4] > 0.0 && th[4] <= 1.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: e_axis must lie in (0,1]", (long long)s);
  if (!(th[6] > 0.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: e_scale must be > 0", (long long)s);
  for (int i : {9, 10})
    if (!(th[i] > 0.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: r2 must be > 0", (long long)s);
  for (int i = 19; i < NP; ++i)
    if (!(th[i] > 0.0)) return fail(CELESTE_E_INVALID, "theta[%lld]: c2 must be > 0", (long long)s);
  return CELESTE_OK;
}

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// Host-side packed metadata: one block [images | sources | work items | 4 zeros (the check's flags)], uploaded
// as it is.  It lives in the context's pinned staging buffer (valid until the context packs the next
// batch), or, for the no-allocation entry point, on the process heap.
struct Packed {
  ImgDev* imgs = nullptr;
  SrcDev* srcs = nullptr;
  WorkItem* items = nullptr;
  unsigned char* block = nullptr;
  size_t o_srcs = 0, o_items = 0, o_flag = 0, bytes = 0;   // parts of the block
  // a pixel subsample's items lie in a block of their own, [work items | first rows of the kept blocks]
  bool own_items = false;
  int* kept_rows = nullptr;
  size_t o_kept = 0, items_bytes = 0;
  PriorDev prior;
  ProfDev prof;
  int tstride = 0;
  int n_src = 0, n_img = 0, n_items = 0;
};
typedef std::vector<unsigned char> HostPack;

int check_thetas(const double* th, int64_t n) {
  const int64_t bad = first_failure(n, 20, [&](int64_t s) { return check_theta(th + s * NP, s) == CELESTE_OK; });
  return bad < n ? check_theta(th + bad * NP, bad) : CELESTE_OK;
}

// Rows of a work item: whole 8-row tile rows holding about `chunk` pixels.
int band_rows(const celeste_image& im, int chunk) { return std::max(TILE, (chunk / std::max(1, im.w)) / TILE * TILE); }
int items_of(const celeste_image& im, int chunk) {
  const int band = band_rows(im, chunk);
  return (im.h + band - 1) / band;
}

// What validate_and_pack leaves: everything, all but the work items (a subsample builds its own, calls that
// evaluate no pixels read none), or nothing but the checks and counts.
enum class Pack { kAll, kNoItems, kCheck };

// Checks the batch and packs its metadata in one pass of the host threads, each over whole sources: checks and
// counts, then (the block allocated) the records.
int validate_and_pack(celeste_ctx* ctx, const celeste_batch* b, Packed* P, HostPack* hp = nullptr,
                      Pack what = Pack::kAll) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  if (!b) return fail(CELESTE_E_INVALID, "batch is NULL");
  if (b->n_sources < 1) return fail(CELESTE_E_INVALID, "n_sources must be >= 1");
  if (b->mem_kind != CELESTE_MEM_HOST && b->mem_kind != CELESTE_MEM_DEVICE)
    return fail(CELESTE_E_INVALID, "mem_kind must be CELESTE_MEM_HOST or CELESTE_MEM_DEVICE");
  if (!b->image_offsets || !b->images) return fail(CELESTE_E_INVALID, "image_offsets/images is NULL");
  if (b->image_offsets[0] != 0) return fail(CELESTE_E_INVALID, "image_offsets[0] must be 0");
  for (int s = 0; s < b->n_sources; ++s) {
    if (b->image_offsets[s + 1] < b->image_offsets[s])
      return fail(CELESTE_E_INVALID, "image_offsets must be non-decreasing");
    if (b->image_offsets[s + 1] == b->image_offsets[s])
      return fail(CELESTE_E_INVALID, "source %d has no images", s);
  }
  const int64_t n_img = b->image_offsets[b->n_sources];
  if (n_img > (int64_t)1 << 30) return fail(CELESTE_E_INVALID, "too many images");
  CHK(make_prior(b->prior, &P->prior));
  CHK(make_profiles(b->profiles, &P->prof));
  const int chunk = std::max(64, ctx->chunk_px);
  const int S = b->n_sources;
  P->n_src = S;
  P->n_img = (int)n_img;
  struct Slice {
    int64_t bad = INT64_MAX, items = 0;
    int max_psf = 1;
  };
  Slice sl[TEAM_MAX];
  int rc = CELESTE_OK;
  int64_t bad = INT64_MAX, n_items = 0;
  team(team_size(n_img, what == Pack::kCheck ? 8 : 20), [&](int t, int nt, Barrier& bar) {
    // sources whose first image lies in this thread's share of the images
    const auto first_src = [&](int k) {
      return k == nt ? S : (int)(std::lower_bound(b->image_offsets, b->image_offsets + S, n_img * k / nt) - b->image_offsets);
    };
    const int s0 = first_src(t), s1 = first_src(t + 1);
    Slice me;
    for (int64_t i = b->image_offsets[s0]; i < b->image_offsets[s1]; ++i) {
      if (check_image(b->images[i], i) != CELESTE_OK) {
        me.bad = i;
        break;
      }
      me.max_psf = std::max(me.max_psf, b->images[i].n_psf);
      me.items += items_of(b->images[i], chunk);
    }
    sl[t] = me;
    bar.wait();
    if (t == 0) {
      int max_psf = 1;
      for (int k = 0; k < nt; ++k) {
        bad = std::min(bad, sl[k].bad);
        max_psf = std::max(max_psf, sl[k].max_psf);
        n_items += sl[k].items;
      }
      if (bad == INT64_MAX && n_items > (int64_t)INT32_MAX / 2) rc = fail(CELESTE_E_INVALID, "too many work items");
      P->tstride = table_stride(max_psf, P->prof.n_exp, P->prof.n_dev);
      if (bad == INT64_MAX && rc == CELESTE_OK && what != Pack::kCheck) {
        P->n_items = what == Pack::kAll ? (int)n_items : 0;
        P->o_srcs = align256(sizeof(ImgDev) * n_img);
        P->o_items = P->o_srcs + align256(sizeof(SrcDev) * S);
        P->o_flag = P->o_items + align256(sizeof(WorkItem) * P->n_items);
        P->bytes = P->o_flag + sizeof(int) * 4;
        if (hp) {
          try {
            hp->resize(P->bytes);
          } catch (const std::bad_alloc&) {
            rc = fail(CELESTE_E_NOMEM, "host allocation of %zu bytes failed", P->bytes);
          }
          P->block = hp->data();
        } else {
          rc = ensure_host(ctx->h_meta, P->bytes);
          P->block = as<unsigned char>(ctx->h_meta);
        }
        P->imgs = reinterpret_cast<ImgDev*>(P->block);
        P->srcs = reinterpret_cast<SrcDev*>(P->block + P->o_srcs);
        P->items = reinterpret_cast<WorkItem*>(P->block + P->o_items);
        if (rc == CELESTE_OK) std::memset(P->block + P->o_flag, 0, sizeof(int) * 4);
      }
    }
    bar.wait();
    if (bad != INT64_MAX || rc != CELESTE_OK || what == Pack::kCheck) return;
    int64_t it = 0;
    for (int k = 0; k < t; ++k) it += sl[k].items;
    for (int s = s0; s < s1; ++s) {
      SrcDev sd;
      sd.img_begin = (int)b->image_offsets[s];
      sd.img_end = (int)b->image_offsets[s + 1];
      sd.item_begin = what == Pack::kAll ? (int)it : 0;
      sd.npix = 0;
      for (int64_t i = sd.img_begin; i < sd.img_end; ++i) {
        const celeste_image& im = b->images[i];
        ImgDev& d = P->imgs[i];
        std::memset(&d, 0, sizeof(d));
        d.pix = im.pixels;
        d.nbr_mean = im.nbr_mean;
        d.nbr_var = im.nbr_var;
        d.h = im.h;
        d.w = im.w;
        d.pitch = im.pitch;
        d.nbr_pitch = im.nbr_pitch ? im.nbr_pitch : im.pitch;
        d.band = im.band;
        d.n_psf = im.n_psf;
        d.src = s;
        d.origin[0] = im.origin[0];
        d.origin[1] = im.origin[1];
        for (int k = 0; k < 6; ++k) d.wcs[k] = im.wcs[k];
        d.sky = im.sky;
        d.calib = im.calib;
        for (int k = 0; k < im.n_psf; ++k)
          for (int j = 0; j < 6; ++j) d.psf[k][j] = im.psf[k][j];
        sd.npix += (int64_t)im.h * im.w;
        if (what == Pack::kAll) {
          d.item_begin = (int)it;
          const int band = band_rows(im, chunk);
          for (int r = 0; r < im.h; r += band) P->items[it++] = WorkItem{(int)i, s, r, std::min(im.h, r + band)};
          d.item_end = (int)it;
        }
      }
      sd.item_end = what == Pack::kAll ? (int)it : 0;
      P->srcs[s] = sd;
    }
  });
  if (bad != INT64_MAX) return check_image(b->images[bad], bad);   // again, for its message
  return rc;
}

// Pixel subsample: the work items are rebuilt over the kept 8-row blocks only.  kept_rows
// receives the first row of every kept block (image by image, in row order); an item takes
// up to a band's worth of one image's consecutive list entries (the blocks need not be
// adjacent), and its [row_begin, row_end) indexes kept_rows.  The item ranges of the images
// and sources and the sources' pixel counts follow.  keep / keep_off: host arrays.
int subsample_items(celeste_ctx* ctx, const celeste_batch* b, Packed* P, const uint8_t* keep,
                    const int64_t* keep_off) {
  if (keep_off[0] != 0) return fail(CELESTE_E_INVALID, "keep_off[0] must be 0");
  const int64_t off_bad = first_failure(
      P->n_img, 3, [&](int64_t i) { return keep_off[i + 1] - keep_off[i] == (b->images[i].h + 7) / 8; });
  if (off_bad < P->n_img)
    return fail(CELESTE_E_INVALID, "image %lld: keep_off must give (h + 7) / 8 blocks", (long long)off_bad);
  const int chunk = std::max(64, ctx->chunk_px), S = P->n_src;
  const int64_t n_img = P->n_img;
  struct Slice {
    int64_t rows = 0, items = 0;
  };
  Slice sl[TEAM_MAX];
  int rc = CELESTE_OK;
  team(team_size(n_img, 40), [&](int t, int nt, Barrier& bar) {
    const auto first_src = [&](int k) {
      return k == nt ? S : (int)(std::lower_bound(b->image_offsets, b->image_offsets + S, n_img * k / nt) - b->image_offsets);
    };
    const int s0 = first_src(t), s1 = first_src(t + 1);
    const auto blocks_per_item = [&](const celeste_image& im) { return band_rows(im, chunk) / TILE; };
    Slice me;
    for (int64_t i = b->image_offsets[s0]; i < b->image_offsets[s1]; ++i) {
      const uint8_t* k = keep + keep_off[i];
      const int nb = (b->images[i].h + 7) / 8, per = blocks_per_item(b->images[i]);
      int64_t n = 0;
      for (int j = 0; j < nb; ++j) n += k[j] ? 1 : 0;
      me.rows += n;
      me.items += (n + per - 1) / per;
    }
    sl[t] = me;
    bar.wait();
    Slice base;
    for (int k = 0; k < t; ++k) {
      base.rows += sl[k].rows;
      base.items += sl[k].items;
    }
    if (t == 0) {
      Slice all;
      for (int k = 0; k < nt; ++k) {
        all.rows += sl[k].rows;
        all.items += sl[k].items;
      }
      P->o_kept = align256(sizeof(WorkItem) * (size_t)all.items);
      P->items_bytes = P->o_kept + sizeof(int) * (size_t)all.rows;
      if (all.rows > (int64_t)INT32_MAX / 2)
        rc = fail(CELESTE_E_INVALID, "too many kept blocks");
      else if (all.items > (int64_t)INT32_MAX / 2)
        rc = fail(CELESTE_E_INVALID, "too many work items");
      else
        rc = ensure_host(ctx->h_items, P->items_bytes);
      P->items = as<WorkItem>(ctx->h_items);
      P->kept_rows = reinterpret_cast<int*>(as<unsigned char>(ctx->h_items) + P->o_kept);
      P->own_items = true;
      P->n_items = (int)all.items;
    }
    bar.wait();
    if (rc != CELESTE_OK) return;
    int64_t row = base.rows, it = base.items;
    for (int s = s0; s < s1; ++s) {
      SrcDev& sd = P->srcs[s];
      sd.npix = 0;
      sd.item_begin = (int)it;
      for (int i = sd.img_begin; i < sd.img_end; ++i) {
        const celeste_image& im = b->images[i];
        const uint8_t* k = keep + keep_off[i];
        const int nb = (im.h + 7) / 8, per = blocks_per_item(im);
        ImgDev& d = P->imgs[i];
        const int64_t first = row;
        for (int j = 0; j < nb; ++j)
          if (k[j]) {
            P->kept_rows[row++] = TILE * j;
            sd.npix += (int64_t)(std::min(im.h, TILE * (j + 1)) - TILE * j) * im.w;
          }
        d.item_begin = (int)it;
        for (int64_t e = first; e < row; e += per)
          P->items[it++] = WorkItem{i, d.src, (int)e, (int)std::min<int64_t>(row, e + per)};
        d.item_end = (int)it;
      }
      sd.item_end = (int)it;
    }
  });
  return rc;
}

// Host data on its way to or from the device goes through two pinned pieces taking turns, so that one is packed (or
// emptied) while the other is copied.  A copy costs about 10 us beside its bytes, so that pieces of 1 MB are the best
// for a few MB; but the first use of pinned memory costs 0.37 us a KB, its pages being mapped one by one, which
// made a context's first call on 100 sources' pixels (3.5 MB) take 1,430 us with one pinned buffer
// for all of them (670 us through pageable memory).  So the pieces begin with 256 KB each, or a 32nd of a
// large transfer, and while a call waits for its kernels it maps more of the ring, which the next calls use:
// 640 us for the first, 330 us in steady state (370 with one buffer, 420 pageable).
constexpr size_t PIECE_MIN = (size_t)256 << 10, PIECE_MAX = (size_t)4 << 20;

// The ring for a transfer of `bytes`, its pieces free: *piece bytes each, the second behind the first.  Where it exists
// and is small, it is made larger only if `grow`.
int ring_for(celeste_ctx* ctx, size_t bytes, bool grow, size_t* piece) {
  for (int k = 0; k < 2; ++k) {
    if (!ctx->ring_ev[k]) HIPCHK(hipEventCreateWithFlags(&ctx->ring_ev[k], hipEventDisableTiming));
    if (ctx->ring_used[k]) HIPCHK(hipEventSynchronize(ctx->ring_ev[k]));   // (left by a call that failed)
    ctx->ring_used[k] = false;
  }
  size_t p = bytes <= 2 * PIECE_MIN ? PIECE_MIN : 4 * PIECE_MIN;
  while (p < PIECE_MAX && p * 4 < bytes) p *= 2;
  if (2 * p > ctx->h_ring.cap && (grow || !ctx->h_ring.p)) {
    if (ctx->h_ring.p) (void)hipHostFree(ctx->h_ring.p);
    ctx->h_ring = DevBuf{};
    ctx->ring_mapped = 0;
    CHK(ensure_host(ctx->h_ring, 2 * p));
  }
  const size_t most = std::min(PIECE_MAX, ctx->h_ring.cap / 2 & ~(size_t)4095);
  const size_t least = std::max(PIECE_MIN, std::min(most, bytes / 32 & ~(size_t)4095));
  *piece = bytes <= 2 * PIECE_MIN ? 2 * PIECE_MIN : std::max(least, ctx->ring_mapped / 2 & ~(size_t)4095);
  ctx->ring_mapped = std::max(ctx->ring_mapped, std::min(bytes, 2 * least));
  return CELESTE_OK;
}

// Maps more of the ring for as long as the stream has work, where the context moves more than 256 KB: pixels, or the
// results of `bytes`.
void ring_map_more(celeste_ctx* ctx, size_t bytes, hipStream_t st) {
  const volatile unsigned char* p = as<unsigned char>(ctx->h_ring);
  if (ctx->ring_mapped < 2 * PIECE_MIN && bytes <= PIECE_MIN) return;
  while (ctx->ring_mapped < ctx->h_ring.cap && hipStreamQuery(st) == hipErrorNotReady) {
    (void)hipGetLastError();   // "not ready" is no error of a later launch
    for (int k = 0; k < 8 && ctx->ring_mapped < ctx->h_ring.cap; ++k, ctx->ring_mapped += 4096) (void)p[ctx->ring_mapped];
  }
  ctx->ring_mapped = std::min(ctx->ring_mapped, ctx->h_ring.cap);   // (it need not begin at a page)
}

int ring_mark(celeste_ctx* ctx, int k, hipStream_t st) {
  HIPCHK(hipEventRecord(ctx->ring_ev[k], st));
  ctx->ring_used[k] = true;
  return CELESTE_OK;
}

int ring_wait(celeste_ctx* ctx, int k) {
  if (ctx->ring_used[k]) HIPCHK(hipEventSynchronize(ctx->ring_ev[k]));
  ctx->ring_used[k] = false;
  return CELESTE_OK;
}

// A host array of h rows of w 4-byte elements, `pitch` elements apart, that goes to element `off` of a device buffer.
struct Part {
  const void* src;
  size_t pitch, off;
  int h, w;
};

// Copies the parts, in the order of their offsets and without gaps, to dst (`total` elements).  The copies are in the
// stream when this returns.
int ring_upload(celeste_ctx* ctx, const std::vector<Part>& parts, size_t total, void* dst, hipStream_t st) {
  size_t piece;
  CHK(ring_for(ctx, 4 * total, true, &piece));
  piece /= 4;
  const int n_pieces = (int)((total + piece - 1) / piece);
  int rc = CELESTE_OK;             // the calling thread's
  bool stop[2] = {false, false};   // whether it failed, as all threads see it behind piece q's barrier: stop[q & 1]
  team(team_size((int64_t)(total / 1024), 60), [&](int t, int nt, Barrier& bar) {   // a thread packs 4 MB in 60 us
    for (int q = 0; q < n_pieces; ++q) {
      const size_t p0 = q * piece, n = std::min(total - p0, piece);
      unsigned char* buf = as<unsigned char>(ctx->h_ring) + (q & 1) * 4 * piece;
      const size_t a = p0 + n * t / nt, e = p0 + n * (t + 1) / nt;   // this thread's elements
      size_t k = std::upper_bound(parts.begin(), parts.end(), a, [](size_t v, const Part& p) { return v < p.off; }) -
                 parts.begin() - 1;
      for (size_t at = a; at < e; ++k) {
        const Part& p = parts[k];
        const size_t end = std::min(e, p.off + (size_t)p.h * p.w), r = (at - p.off) / p.w;
        const unsigned char* row = static_cast<const unsigned char*>(p.src) + 4 * r * p.pitch;
        for (size_t c = (at - p.off) - r * p.w; at < end; c = 0, row += 4 * p.pitch) {
          const size_t m = std::min(end - at, (size_t)p.w - c);
          std::memcpy(buf + 4 * (at - p0), row + 4 * c, 4 * m);
          at += m;
        }
      }
      if (t == 0) {
        if (rc == CELESTE_OK && q + 1 < n_pieces) rc = ring_wait(ctx, (q + 1) & 1);
        stop[q & 1] = rc != CELESTE_OK;
      }
      bar.wait();   // the piece is packed, and the next one free
      if (stop[q & 1]) return;
      if (t == 0) {
        const hipError_t err = hipMemcpyAsync(static_cast<unsigned char*>(dst) + 4 * p0, buf, 4 * n, hipMemcpyHostToDevice, st);
        rc = err != hipSuccess ? fail(CELESTE_E_DEVICE, "copy to the device: %s", hipGetErrorString(err))
             : n_pieces > 1   ? ring_mark(ctx, q & 1, st)
                              : CELESTE_OK;
      }
    }
  });
  return rc;
}

// Copies n doubles from src (device memory) to the host, piece by piece: give(values, first, count).
template <class F>
int ring_download(celeste_ctx* ctx, const double* src, size_t n, hipStream_t st, F give) {
  size_t piece;
  CHK(ring_for(ctx, sizeof(double) * n, false, &piece));
  const size_t per = piece / sizeof(double), n_pieces = (n + per - 1) / per;
  for (size_t q = 0; q <= n_pieces; ++q) {
    if (q < n_pieces) {
      HIPCHK(hipMemcpyAsync(as<unsigned char>(ctx->h_ring) + (q & 1) * piece, src + q * per,
                            sizeof(double) * std::min(per, n - q * per), hipMemcpyDeviceToHost, st));
      CHK(ring_mark(ctx, q & 1, st));
    }
    if (q == 0) continue;
    const size_t at = (q - 1) * per;
    CHK(ring_wait(ctx, (q - 1) & 1));
    give(reinterpret_cast<const double*>(as<unsigned char>(ctx->h_ring) + ((q - 1) & 1) * piece), at, std::min(per, n - at));
  }
  return CELESTE_OK;
}

// Copies host pixel arrays into one device staging buffer and repoints the images.
int stage_host_pixels(celeste_ctx* ctx, const celeste_batch* b, Packed* P, hipStream_t st) {
  std::vector<Part> parts;
  parts.reserve((size_t)P->n_img);
  size_t total = 0;
  for (int i = 0; i < P->n_img; ++i) {
    const celeste_image& im = b->images[i];
    const float* srcs[3] = {im.pixels, im.nbr_mean, im.nbr_var};
    for (int k = 0; k < 3; ++k) {
      if (!srcs[k]) continue;
      const int pitch = k == 0 || !im.nbr_pitch ? im.pitch : im.nbr_pitch;
      const bool gaps = pitch != im.w;   // rows without them are packed as one
      parts.push_back(Part{srcs[k], (size_t)pitch, total, gaps ? im.h : 1, gaps ? im.w : im.h * im.w});
      total += (size_t)im.h * im.w;
    }
  }
  CHK(ensure(ctx->staging, total * sizeof(float)));
  float* base = as<float>(ctx->staging);
  CHK(ring_upload(ctx, parts, total, base, st));
  size_t k = 0;
  for (int i = 0; i < P->n_img; ++i) {
    const celeste_image& im = b->images[i];
    ImgDev& d = P->imgs[i];
    d.pitch = d.w;
    d.nbr_pitch = d.w;
    d.pix = base + parts[k++].off;
    d.nbr_mean = im.nbr_mean ? base + parts[k++].off : nullptr;
    d.nbr_var = im.nbr_var ? base + parts[k++].off : nullptr;
  }
  return CELESTE_OK;
}

// Device buffers of one evaluation: packed metadata, setup tables, per-item partial sums,
// per-image constants, the pixel-check flag and the log n! table.
struct EvalBufs {
  ImgDev* imgs = nullptr;
  WorkItem* items = nullptr;
  SrcDev* srcs = nullptr;
  double* img_const = nullptr;
  float* tables = nullptr;
  double* partials = nullptr;
  int* flag = nullptr;
  double* lfact = nullptr;
  bool lfact_ready = false;   // the table holds its values (else it is filled before use)
  // the parts of the metadata block, copied to base
  void place(const Packed& P, unsigned char* base) {
    imgs = reinterpret_cast<ImgDev*>(base);
    srcs = reinterpret_cast<SrcDev*>(base + P.o_srcs);
    items = reinterpret_cast<WorkItem*>(base + P.o_items);
    flag = reinterpret_cast<int*>(base + P.o_flag);
  }
};

// The context's own buffers, grown to the batch.
int ctx_bufs(celeste_ctx* ctx, const Packed* P, EvalBufs* B) {
  CHK(ensure(ctx->meta, P->bytes));
  if (P->own_items) CHK(ensure(ctx->items_kept, P->items_bytes));
  CHK(ensure(ctx->img_const, sizeof(double) * P->n_img));
  CHK(ensure(ctx->tables, sizeof(float) * (size_t)P->tstride * P->n_img));
  CHK(ensure(ctx->partials, sizeof(double) * (size_t)NACC * P->n_items));
  if (!ctx->lfact_ready) CHK(ensure(ctx->lfact, sizeof(double) * LFACT_N));
  B->place(*P, as<unsigned char>(ctx->meta));
  if (P->own_items) B->items = as<WorkItem>(ctx->items_kept);
  ctx->imgs.p = B->imgs;
  ctx->srcs.p = B->srcs;
  ctx->items.p = B->items;
  B->img_const = as<double>(ctx->img_const);
  B->tables = as<float>(ctx->tables);
  B->partials = as<double>(ctx->partials);
  B->lfact = as<double>(ctx->lfact);
  B->lfact_ready = ctx->lfact_ready;
  return CELESTE_OK;
}

// The metadata into the buffers B (host batches' pixels are staged first), and, where the call reads pixels, the
// launch of their check and of the per-image constants.  Nothing here waits: B.flag tells once the stream has run
// (FLAG_PIXELS, and FLAG_THETA where theta, device memory, is given to be checked).
int upload_in(celeste_ctx* ctx, const celeste_batch* b, Packed* P, EvalBufs* B, hipStream_t st, bool pixels,
              const double* theta = nullptr) {
  if (b->mem_kind == CELESTE_MEM_HOST) CHK(stage_host_pixels(ctx, b, P, st));
  HIPCHK(hipMemcpyAsync(B->imgs, P->block, P->bytes, hipMemcpyHostToDevice, st));
  if (P->own_items && P->n_items > 0)
    HIPCHK(hipMemcpyAsync(B->items, P->items, P->items_bytes, hipMemcpyHostToDevice, st));
  if (!pixels) return CELESTE_OK;
  if (!B->lfact_ready) {
    HIPCHK(launch_lfact(B->lfact, st));
    B->lfact_ready = true;   // complete before first use, on this stream and, once the call has waited, on every other
  }
  HIPCHK(launch_check_const(B->imgs, P->n_img, B->lfact, B->img_const, B->flag, st, theta, theta ? P->n_src : 0));
  return CELESTE_OK;
}

// The error of estimates (device memory) of which the device found one out of range.
int theta_error(const double* theta, size_t n, hipStream_t st) {
  std::vector<double> h(NP * n);
  HIPCHK(hipMemcpyAsync(h.data(), theta, sizeof(double) * NP * n, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  CHK(check_thetas(h.data(), (int64_t)n));
  return fail(CELESTE_E_INVALID, "theta out of range");
}

int pixel_error() { return fail(CELESTE_E_INVALID, "pixel or neighbour arrays hold negative or non-finite values"); }

// upload_in on the context's own buffers; waits for the check of the pixels.
int prepare(celeste_ctx* ctx, const celeste_batch* b, Packed* P, hipStream_t st, bool pixels = true) {
  EvalBufs B;
  CHK(ctx_bufs(ctx, P, &B));
  CHK(upload_in(ctx, b, P, &B, st, pixels));
  if (!pixels) return CELESTE_OK;
  int bad = 0;
  HIPCHK(hipMemcpyAsync(&bad, B.flag, sizeof(int), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  ctx->lfact_ready = ctx->lfact_ready || B.lfact_ready;
  return bad ? pixel_error() : CELESTE_OK;
}

hipStream_t pick(celeste_ctx* ctx, void* stream) { return stream ? (hipStream_t)stream : ctx->stream; }

unsigned long long* ctr_full(celeste_ctx* c) { return as<unsigned long long>(c->ctr); }
unsigned long long* ctr_value(celeste_ctx* c) { return as<unsigned long long>(c->ctr) + 1; }
unsigned long long* ctr_grad(celeste_ctx* c) { return as<unsigned long long>(c->ctr) + 2; }
// counters [3, 9) belong to the trust-region subproblem (FitParams::tr_ctr)
unsigned long long* ctr_trial(celeste_ctx* c) { return as<unsigned long long>(c->ctr) + 9; }
unsigned long long* ctr_taken(celeste_ctx* c) { return as<unsigned long long>(c->ctr) + 10; }
constexpr int N_CTR = 11;

// HIP events between the kernel phases of one iteration (profile mode).
struct PhaseTimer {
  bool on = false;
  hipEvent_t ev[9] = {};
  int init(bool enable) {
    on = enable;
    if (!on) return CELESTE_OK;
    for (auto& e : ev) HIPCHK(hipEventCreate(&e));
    return CELESTE_OK;
  }
  ~PhaseTimer() {
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
  }
  void mark(int k, hipStream_t st) {
    if (on) (void)hipEventRecord(ev[k], st);
  }
  float span(int a, int b) {
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, ev[a], ev[b]);
    return ms;
  }
};

int eval_impl(celeste_ctx* ctx, const celeste_batch* b, const double* theta, double* elbo, double* grad,
              double* hess, void* stream, const uint8_t* keep, const int64_t* keep_off, double keep_prob,
              bool noalloc = false);
int scratch_init(int device);

}  // namespace

// =============================================================================== ABI

extern "C" {

const char* celeste_last_error(void) { return g_err.c_str(); }

void celeste_fit_opts_default(celeste_fit_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->max_iter = 50;
  o->init_mode = CELESTE_INIT_AS_GIVEN;
  o->pred_rtol = 1e-8;
  o->curv_tol = 1e-8;
  o->delta0 = 1.0;
  o->delta_max = 100.0;
  o->delta_min = 1e-10;
  o->eta = 0.1;
  o->u_box = 3.0;
  o->poll_every = 4;
}

int celeste_ctx_create(int hip_device, celeste_ctx** out) {
  if (!out) return fail(CELESTE_E_INVALID, "out is NULL");
  *out = nullptr;
  int n = 0;
  HIPCHK(hipGetDeviceCount(&n));
  if (hip_device < 0 || hip_device >= n) return fail(CELESTE_E_INVALID, "device %d not in 0..%d", hip_device, n - 1);
  HIPCHK(hipSetDevice(hip_device));
  celeste_ctx* c = new (std::nothrow) celeste_ctx();
  if (!c) return fail(CELESTE_E_NOMEM, "context allocation failed");
  c->device = hip_device;
  if (hipDeviceGetAttribute(&c->n_cu, hipDeviceAttributeMultiprocessorCount, hip_device) != hipSuccess ||
      c->n_cu < 1)
    c->n_cu = 256;
  if (scratch_init(hip_device) != CELESTE_OK) {   // device address of the no-allocation scratch
    delete c;
    return CELESTE_E_DEVICE;
  }
  if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess) {
    delete c;
    return fail(CELESTE_E_DEVICE, "stream creation failed");
  }
  if (ensure(c->ctr, N_CTR * sizeof(unsigned long long)) != CELESTE_OK ||
      hipMemset(c->ctr.p, 0, N_CTR * sizeof(unsigned long long)) != hipSuccess) {
    (void)hipStreamDestroy(c->stream);
    if (c->ctr.p) (void)hipFree(c->ctr.p);
    delete c;
    return fail(CELESTE_E_DEVICE, "counter allocation failed");
  }
  {
    // Exact-zero threshold: where the device's exp2 returns exactly 0 below 2^-126 (results
    // that would be subnormal are flushed), a component whose log2 density is below -127 on a
    // whole tile contributes exactly 0 and the threshold is -127; otherwise -160 (below the
    // smallest subnormal).
    const float in[4] = {-126.5f, -127.0f, -135.0f, -149.5f};
    float res[4] = {1.f, 1.f, 1.f, 1.f};
    DevBuf pb;
    if (ensure(pb, sizeof(in) * 2) == CELESTE_OK) {
      float* d = as<float>(pb);
      if (hipMemcpy(d, in, sizeof(in), hipMemcpyHostToDevice) == hipSuccess &&
          launch_exp2_probe(d, d + 4, 4, c->stream) == hipSuccess &&
          hipMemcpyAsync(res, d + 4, sizeof(res), hipMemcpyDeviceToHost, c->stream) == hipSuccess &&
          hipStreamSynchronize(c->stream) == hipSuccess)
        c->exp2_flushes = res[0] == 0.f && res[1] == 0.f && res[2] == 0.f && res[3] == 0.f;
      c->e_zero = c->exp2_flushes ? -127.f : -160.f;
      (void)hipFree(pb.p);
    }
  }
  *out = c;
  return CELESTE_OK;
}

int celeste_ctx_get_stats(celeste_ctx* c, celeste_stats* out, int reset) {
  if (!c || !out) return fail(CELESTE_E_INVALID, "context and out must not be NULL");
  HIPCHK(hipSetDevice(c->device));
  unsigned long long h[N_CTR] = {};
  HIPCHK(hipMemcpy(h, c->ctr.p, sizeof(h), hipMemcpyDeviceToHost));
  c->stats.full_px = (int64_t)(h[0] + h[9]);
  c->stats.trial_full_px = (int64_t)h[9];
  c->stats.taken_px = (int64_t)h[10];
  c->stats.value_px = (int64_t)h[1];
  c->stats.grad_px = (int64_t)h[2];
  c->stats.tr_interior = (int64_t)h[3];
  c->stats.tr_boundary = (int64_t)h[4];
  c->stats.tr_eigen = (int64_t)h[5];
  c->stats.tr_sweeps = (int64_t)h[6];
  c->stats.tr_sweep_cap = (int64_t)h[7];
  c->stats.tr_newton_steps = (int64_t)h[8];
  *out = c->stats;
  if (reset) {
    HIPCHK(hipMemset(c->ctr.p, 0, sizeof(h)));
    c->stats = celeste_stats{};
  }
  return CELESTE_OK;
}

void celeste_ctx_destroy(celeste_ctx* c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  (void)hipStreamSynchronize(c->stream);
  DevBuf* bufs[] = {&c->meta, &c->items_kept, &c->tables, &c->partials, &c->img_const, &c->staging,
                    &c->theta, &c->o_elbo, &c->st_buf, &c->ctr, &c->sur,
                    &c->tile_off, &c->img_field, &c->nbr_off, &c->tables2, &c->fsky, &c->theta_flag,
                    &c->lr_in, &c->lr_cov, &c->lr_status, &c->lr_eval,
                    &c->lfact, &c->lb_buf, &c->imgs_s, &c->items_s, &c->srcs_s, &c->partials_s, &c->qbuf};
  for (DevBuf* b : bufs)
    if (b->p) (void)hipFree(b->p);
  for (DevBuf* b : {&c->h_meta, &c->h_items, &c->h_lists, &c->h_poll, &c->h_flags, &c->h_ring})
    if (b->p) (void)hipHostFree(b->p);
  for (hipEvent_t e : c->ring_ev)
    if (e) (void)hipEventDestroy(e);
  (void)hipStreamDestroy(c->stream);
  delete c;
}

int celeste_ctx_set_option(celeste_ctx* c, int option, int64_t value) {
  if (!c) return fail(CELESTE_E_INVALID, "context is NULL");
  switch (option) {
    case CELESTE_OPT_CHUNK_PX:
      if (value < 64 || value > (1 << 24)) return fail(CELESTE_E_INVALID, "chunk_px must be in 64..2^24");
      c->chunk_px = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_BLOCK:
      if (value != 128 && value != 256) return fail(CELESTE_E_INVALID, "block must be 128 or 256");
      c->block = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_USE_GRAPH:
      c->use_graph = value ? 1 : 0;
      return CELESTE_OK;
    case CELESTE_OPT_PROFILE:
      c->profile = value ? 1 : 0;
      return CELESTE_OK;
    case CELESTE_OPT_VARIANT:
      if (value < 0 || value > 7) return fail(CELESTE_E_INVALID, "variant must be in 0..7");
      c->variant = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_TILE_W:
    case CELESTE_OPT_VALUE_TILE_W: {
      int l = -1;
      for (int k = 3; k <= 6; ++k)
        if (value == (1 << k)) l = k;
      if (l < 0) return fail(CELESTE_E_INVALID, "tile width must be 8, 16, 32 or 64");
      (option == CELESTE_OPT_TILE_W ? c->tile_log2 : c->vtile_log2) = l;
      return CELESTE_OK;
    }
    case CELESTE_OPT_VALUE_BLOCK:
      if (value != 128 && value != 256) return fail(CELESTE_E_INVALID, "value block must be 128 or 256");
      c->vblock = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_PERSISTENT:
      if (value < -1 || value > 16)
        return fail(CELESTE_E_INVALID, "persistent blocks per compute unit must be -1..16");
      c->persistent = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_FP64_SUMS:
      if (value != 0 && value != 1) return fail(CELESTE_E_INVALID, "FP64 sums must be 0 or 1");
      c->fp64_sums = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_TRIAL_DERIVATIVES:
      if (value != 0 && value != 1) return fail(CELESTE_E_INVALID, "trial derivatives must be 0 or 1");
      c->trial_derivs = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_TR_CHOLESKY:
      if (value != 0 && value != 1) return fail(CELESTE_E_INVALID, "trust-region Cholesky path must be 0 or 1");
      c->tr_chol = (int)value;
      return CELESTE_OK;
    case CELESTE_OPT_EXACT_ZERO:
      if (value != 0 && value != 1 && value != 127 && value != 160)
        return fail(CELESTE_E_INVALID, "exact-zero threshold must be 0, 1, 127 or 160");
      if (value == 127 && !c->exp2_flushes)
        return fail(CELESTE_E_UNSUPPORTED, "this device's exp2 does not flush results below 2^-126");
      if (value == 1)
        c->e_zero = -INFINITY;   // every skip test (log2 density >= threshold) passes: nothing is skipped
      else
        c->e_zero = value == 160 || (value == 0 && !c->exp2_flushes) ? -160.f : -127.f;
      return CELESTE_OK;
    default:
      return fail(CELESTE_E_INVALID, "unknown option %d", option);
  }
}

size_t celeste_struct_size(int which) {
  switch (which) {
    case 0: return sizeof(celeste_image);
    case 1: return sizeof(celeste_prior);
    case 2: return sizeof(celeste_profiles);
    case 3: return sizeof(celeste_batch);
    case 4: return sizeof(celeste_fit_opts);
    case 5: return sizeof(celeste_fit_result);
    case 6: return sizeof(celeste_stats);
    case 7: return sizeof(celeste_tune_result);
    case 8: return sizeof(celeste_lbfgs_opts);
    default: return 0;
  }
}

int celeste_elbo_eval(celeste_ctx* ctx, const celeste_batch* b, const double* theta, double* elbo, double* grad,
                      double* hess, void* stream) {
  return eval_impl(ctx, b, theta, elbo, grad, hess, stream, nullptr, nullptr, 1.0);
}

int celeste_elbo_eval_noalloc(celeste_ctx* ctx, const celeste_batch* b, const double* theta, double* elbo,
                              double* grad, double* hess, void* stream) {
  return eval_impl(ctx, b, theta, elbo, grad, hess, stream, nullptr, nullptr, 1.0, true);
}

int celeste_elbo_eval_sampled(celeste_ctx* ctx, const celeste_batch* b, const double* theta, const uint8_t* keep,
                              const int64_t* keep_off, double keep_prob, double* elbo, double* grad, double* hess,
                              void* stream) {
  if (!keep || !keep_off) return fail(CELESTE_E_INVALID, "keep and keep_off must not be NULL");
  if (!(keep_prob > 0.0 && keep_prob <= 1.0)) return fail(CELESTE_E_INVALID, "keep_prob must be in (0, 1]");
  return eval_impl(ctx, b, theta, elbo, grad, hess, stream, keep, keep_off, keep_prob);
}

int celeste_lr_covariance_from_hessian(celeste_ctx* ctx, int64_t n, int mem_kind, const double* theta,
                                       const double* u0, double u_box, const double* grad, const double* hess,
                                       double* cov, int32_t* status, void* stream) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  if (n < 0 || n > (int64_t)INT32_MAX / 2) return fail(CELESTE_E_INVALID, "n out of range");
  if (mem_kind != CELESTE_MEM_HOST && mem_kind != CELESTE_MEM_DEVICE)
    return fail(CELESTE_E_INVALID, "mem_kind must be CELESTE_MEM_HOST or CELESTE_MEM_DEVICE");
  if (!theta || !u0 || !grad || !hess || !cov || !status) return fail(CELESTE_E_INVALID, "NULL argument");
  if (!(u_box > 0.0) || !std::isfinite(u_box)) return fail(CELESTE_E_INVALID, "u_box must be finite and > 0");
  if (n == 0) return CELESTE_OK;
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = pick(ctx, stream);
  const size_t S = (size_t)n;
  const double *d_th = theta, *d_u0 = u0, *d_g = grad, *d_h = hess;
  double* d_cov = cov;
  if (mem_kind == CELESTE_MEM_HOST) {
    CHK(ensure(ctx->lr_in, sizeof(double) * S * (NP + 2 + NP + NP * NP)));
    double* base = as<double>(ctx->lr_in);
    double *th = base, *uu = th + S * NP, *gg = uu + S * 2, *hh = gg + S * NP;
    HIPCHK(hipMemcpyAsync(th, theta, sizeof(double) * S * NP, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(uu, u0, sizeof(double) * S * 2, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(gg, grad, sizeof(double) * S * NP, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(hh, hess, sizeof(double) * S * NP * NP, hipMemcpyHostToDevice, st));
    d_th = th;
    d_u0 = uu;
    d_g = gg;
    d_h = hh;
    CHK(ensure(ctx->lr_cov, sizeof(double) * S * NP * NP));
    d_cov = as<double>(ctx->lr_cov);
  }
  CHK(ensure(ctx->lr_status, sizeof(int) * S));
  PhaseTimer T;
  CHK(T.init(ctx->profile != 0));
  T.mark(0, st);
  HIPCHK(launch_lr_cov(d_th, d_u0, u_box, d_g, d_h, (int)S, d_cov, as<int>(ctx->lr_status), st));
  T.mark(1, st);
  if (mem_kind == CELESTE_MEM_HOST)
    HIPCHK(hipMemcpyAsync(cov, d_cov, sizeof(double) * S * NP * NP, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(status, ctx->lr_status.p, sizeof(int32_t) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  ctx->stats.lr_launches += 1;
  if (T.on) ctx->stats.ms_lr += T.span(0, 1);
  return CELESTE_OK;
}

int celeste_lr_covariance(celeste_ctx* ctx, const celeste_batch* b, const double* theta, const double* u0,
                          double u_box, double* cov, int32_t* status, void* stream) {
  if (!ctx || !b) return fail(CELESTE_E_INVALID, "context or batch is NULL");
  if (!theta || !u0 || !cov || !status) return fail(CELESTE_E_INVALID, "NULL argument");
  if (b->n_sources < 1) return fail(CELESTE_E_INVALID, "n_sources must be >= 1");
  if (!(u_box > 0.0) || !std::isfinite(u_box)) return fail(CELESTE_E_INVALID, "u_box must be finite and > 0");
  const size_t S = (size_t)b->n_sources;
  if (b->mem_kind == CELESTE_MEM_HOST) {
    std::vector<double> e(S), g(S * NP), h(S * NP * NP);
    CHK(eval_impl(ctx, b, theta, e.data(), g.data(), h.data(), stream, nullptr, nullptr, 1.0));
    return celeste_lr_covariance_from_hessian(ctx, (int64_t)S, CELESTE_MEM_HOST, theta, u0, u_box, g.data(),
                                              h.data(), cov, status, stream);
  }
  CHK(ensure(ctx->lr_eval, sizeof(double) * S * (1 + NP + NP * NP)));
  double* e = as<double>(ctx->lr_eval);
  double* g = e + S;
  double* h = g + S * NP;
  CHK(eval_impl(ctx, b, theta, e, g, h, stream, nullptr, nullptr, 1.0));
  return celeste_lr_covariance_from_hessian(ctx, (int64_t)S, CELESTE_MEM_DEVICE, theta, u0, u_box, g, h, cov, status,
                                            stream);
}

}  // extern "C"

namespace {

int scratch_bufs(celeste_ctx* ctx, const Packed* P, int per_item, EvalBufs* B);
void scratch_lfact_filled(int device);

int eval_impl(celeste_ctx* ctx, const celeste_batch* b, const double* theta, double* elbo, double* grad,
              double* hess, void* stream, const uint8_t* keep, const int64_t* keep_off, double keep_prob,
              bool noalloc) {
  Packed P;
  HostPack hp;
  CHK(validate_and_pack(ctx, b, &P, noalloc ? &hp : nullptr, keep ? Pack::kNoItems : Pack::kAll));
  if (!theta || !elbo) return fail(CELESTE_E_INVALID, "theta and elbo must not be NULL");
  if (hess && !grad) return fail(CELESTE_E_INVALID, "hess requires grad");
  const bool on_host = b->mem_kind == CELESTE_MEM_HOST;
  if (noalloc && on_host)
    return fail(CELESTE_E_INVALID, "the no-allocation evaluation takes device batches only (mem_kind DEVICE)");
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = pick(ctx, stream);
  const size_t S = P.n_src;
  // The checks of pixels and of estimates on the device run in the same stream as the evaluation, whose reductions
  // write nothing once one has failed; one wait at the end tells (with a wait after each check, one source's
  // evaluation took 154 us instead of 115).  A subsample's list is checked on the host
  // after the estimates, so there they are read back first.
  const double* th_dev = theta;
  const bool check_on_device = !on_host && !keep;
  std::vector<double> th_host;
  if (on_host) {
    CHK(check_thetas(theta, (int64_t)S));
    CHK(ensure(ctx->theta, sizeof(double) * NP * S));
    HIPCHK(hipMemcpyAsync(ctx->theta.p, theta, sizeof(double) * NP * S, hipMemcpyHostToDevice, st));
    th_dev = as<double>(ctx->theta);
  } else if (keep) {
    th_host.resize(NP * S);
    HIPCHK(hipMemcpyAsync(th_host.data(), theta, sizeof(double) * NP * S, hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    CHK(check_thetas(th_host.data(), (int64_t)S));
  }
  double px_weight = 1.0;
  if (keep) {
    CHK(subsample_items(ctx, b, &P, keep, keep_off));
    px_weight = 1.0 / keep_prob;
  }
  EvalBufs B;
  if (noalloc)
    CHK(scratch_bufs(ctx, &P, grad ? (hess ? NACC : NGRAD) : 1, &B));
  else
    CHK(ctx_bufs(ctx, &P, &B));
  const int* kept = keep ? reinterpret_cast<int*>(as<unsigned char>(ctx->items_kept) + P.o_kept) : nullptr;
  // results of a host batch: one device block, read back through the ring
  const size_t n_out = S * (1 + (grad ? NP : 0) + (hess ? NP * NP : 0));
  double *d_elbo = elbo, *d_grad = grad, *d_hess = hess;
  if (on_host) {
    CHK(ensure(ctx->o_elbo, sizeof(double) * n_out));
    d_elbo = as<double>(ctx->o_elbo);
    if (grad) d_grad = d_elbo + S;
    if (hess) d_hess = d_grad + S * NP;
  }
  CHK(upload_in(ctx, b, &P, &B, st, true, check_on_device ? th_dev : nullptr));
  PhaseTimer T;
  CHK(T.init(ctx->profile != 0 && !noalloc));   // events are not created on the no-allocation path
  T.mark(0, st);
  HIPCHK(launch_setup(B.imgs, P.n_img, th_dev, nullptr, P.prof, B.tables, P.tstride, st, grad != nullptr));
  T.mark(1, st);
  int64_t* launches = nullptr;
  if (grad && hess) {
    HIPCHK(launch_eval_full(B.items, P.n_items, B.imgs, B.tables, P.tstride, P.prof.n_exp, P.prof.n_dev, nullptr,
                            B.partials, ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st, kept));
    T.mark(2, st);
    HIPCHK(launch_reduce_full(B.srcs, P.n_src, B.imgs, B.partials, B.img_const, th_dev, P.prior, nullptr, d_elbo,
                              d_grad, d_hess, ctr_full(ctx), st, px_weight, B.flag));
    launches = &ctx->stats.full_launches;
  } else if (grad) {
    HIPCHK(launch_eval_grad(B.items, P.n_items, B.imgs, B.tables, P.tstride, P.prof.n_exp, P.prof.n_dev, nullptr,
                            B.partials, ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st, kept));
    T.mark(2, st);
    HIPCHK(launch_reduce_grad(B.srcs, P.n_src, B.imgs, B.partials, B.img_const, th_dev, P.prior, nullptr, d_elbo,
                              d_grad, ctr_grad(ctx), st, px_weight, B.flag));
    launches = &ctx->stats.grad_launches;
  } else {
    HIPCHK(launch_eval_value(B.items, P.n_items, B.imgs, B.tables, P.tstride, P.prof.n_exp, P.prof.n_dev, nullptr,
                             B.partials, ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st, kept));
    T.mark(2, st);
    HIPCHK(launch_reduce_value(B.srcs, P.n_src, B.imgs, B.partials, B.img_const, th_dev, P.prior, nullptr, d_elbo,
                               ctr_value(ctx), st, px_weight, B.flag));
    launches = &ctx->stats.value_launches;
  }
  T.mark(3, st);
  if (on_host) ring_map_more(ctx, sizeof(double) * n_out, st);
  int bad = 0;
  HIPCHK(hipMemcpyAsync(&bad, B.flag, sizeof(int), hipMemcpyDeviceToHost, st));
  // results that fit in what the ring has used, or in 256 KB of it (it holds at least two such pieces), come with the
  // flag; the pixels' copies out of the ring are ahead in the stream
  const bool one_copy = on_host && sizeof(double) * n_out <= std::max(ctx->ring_mapped, PIECE_MIN);
  if (one_copy) HIPCHK(hipMemcpyAsync(ctx->h_ring.p, d_elbo, sizeof(double) * n_out, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  if (noalloc) {
    if (B.lfact_ready) scratch_lfact_filled(ctx->device);
  } else {
    ctx->lfact_ready = ctx->lfact_ready || B.lfact_ready;
  }
  if (bad & FLAG_THETA) return theta_error(theta, S, st);
  if (bad) return pixel_error();
  *launches += 1;
  if (on_host) {
    // entries [at, at + n) of the results at src to the caller's arrays
    const auto give = [&](const double* src, size_t at, size_t n) {
      const size_t sizes[3] = {S, grad ? S * NP : 0, hess ? S * NP * NP : 0};
      double* const to[3] = {elbo, grad, hess};
      for (size_t k = 0, first = 0; k < 3; first += sizes[k++]) {
        const size_t b0 = std::max(at, first), b1 = std::min(at + n, first + sizes[k]);
        if (b0 < b1) std::memcpy(to[k] + (b0 - first), src + (b0 - at), sizeof(double) * (b1 - b0));
      }
    };
    if (one_copy) {
      give(as<double>(ctx->h_ring), 0, n_out);
    } else if (ctx->ring_mapped >= 2 * PIECE_MIN || sizeof(double) * n_out <= 4 * PIECE_MIN) {
      CHK(ring_download(ctx, d_elbo, n_out, st, give));
    } else {
      // a new ring, or the first use of what there is of one, costs more than pageable copies from about 1 MB: first
      // Hessians of 300 sources of 5 x 5 pixels 400 us, 920 through a ring made for them; 330 and 304 later on
      HIPCHK(hipMemcpyAsync(elbo, d_elbo, sizeof(double) * S, hipMemcpyDeviceToHost, st));
      if (grad) HIPCHK(hipMemcpyAsync(grad, d_grad, sizeof(double) * S * NP, hipMemcpyDeviceToHost, st));
      if (hess) HIPCHK(hipMemcpyAsync(hess, d_hess, sizeof(double) * S * NP * NP, hipMemcpyDeviceToHost, st));
      HIPCHK(hipStreamSynchronize(st));
    }
  }
  if (T.on) {
    ctx->stats.ms_setup += T.span(0, 1);
    (hess ? ctx->stats.ms_full : grad ? ctx->stats.ms_grad : ctx->stats.ms_value) += T.span(1, 2);
    (hess ? ctx->stats.ms_reduce_full : grad ? ctx->stats.ms_reduce_grad : ctx->stats.ms_reduce_value) += T.span(2, 3);
  }
  return CELESTE_OK;
}

}  // namespace

// =============================================================================== no-allocation scratch

// Device memory of celeste_elbo_eval_noalloc: one array on every GPU the library runs on,
// resident from the code object's load until the process ends, shared by every such call on
// that GPU (it keeps the last call's contents, and calls that overlap on one GPU race).  In
// host code the array's name is a host-side stand-in, not a device address: host code uses
// only the per-device address that hipGetSymbolAddress returns (scratch_init).
static __device__ __align__(256) unsigned char scratch[CELESTE_NOALLOC_SCRATCH_BYTES];

namespace {

struct ScratchSlot {
  unsigned char* ptr = nullptr;   // device address of the scratch array on this GPU
  bool lfact_ready = false;       // its log n! region holds the table
};
std::mutex g_scratch_mu;
std::unordered_map<int, ScratchSlot> g_scratch;

// Once per device, with that device current (context creation): the device address of the
// scratch array on it.
int scratch_init(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  ScratchSlot& sl = g_scratch[device];
  if (sl.ptr) return CELESTE_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return fail(CELESTE_E_DEVICE, "address of the scratch array on device %d: %s", device, hipGetErrorString(e));
  }
  sl.ptr = static_cast<unsigned char*>(ptr);
  return CELESTE_OK;
}

// The buffers of one evaluation carved from the device's scratch array: the log n! table
// first (filled once per device, never written by anything else), then the call's own
// regions.  E_NOMEM when the batch does not fit.
int scratch_bufs(celeste_ctx* ctx, const Packed* P, int per_item, EvalBufs* B) {
  ScratchSlot sl;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch.find(ctx->device);
    if (it == g_scratch.end() || !it->second.ptr)
      return fail(CELESTE_E_DEVICE, "no scratch address for device %d", ctx->device);
    sl = it->second;
  }
  size_t off = 0;
  auto carve = [&off](size_t bytes) {
    const size_t o = off;
    off += align256(bytes);
    return o;
  };
  const size_t o_lfact = carve(sizeof(double) * LFACT_N);
  const size_t o_meta = carve(P->bytes);
  const size_t o_const = carve(sizeof(double) * P->n_img);
  const size_t o_tables = carve(sizeof(float) * (size_t)P->tstride * P->n_img);
  const size_t o_part = carve(sizeof(double) * (size_t)per_item * P->n_items);
  if (off > CELESTE_NOALLOC_SCRATCH_BYTES)
    return fail(CELESTE_E_NOMEM,
                "the batch (%d sources, %d images, %d work items) needs %zu bytes of device scratch; "
                "celeste_elbo_eval_noalloc holds at most %zu: split the batch or use celeste_elbo_eval",
                P->n_src, P->n_img, P->n_items, off, (size_t)CELESTE_NOALLOC_SCRATCH_BYTES);
  unsigned char* base = sl.ptr;
  B->lfact = reinterpret_cast<double*>(base + o_lfact);
  B->place(*P, base + o_meta);
  B->img_const = reinterpret_cast<double*>(base + o_const);
  B->tables = reinterpret_cast<float*>(base + o_tables);
  B->partials = reinterpret_cast<double*>(base + o_part);
  B->lfact_ready = sl.lfact_ready;
  return CELESTE_OK;
}

void scratch_lfact_filled(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  g_scratch[device].lfact_ready = true;
}

}  // namespace

// =============================================================================== fits

namespace {

struct FitBufs {
  FitDev d;
};

int alloc_fit(celeste_ctx* ctx, int S, FitDev* f) {
  const size_t nd = (size_t)S * (NP * 6 + 3 * NP * NP + 2 + 7);
  const size_t ni = (size_t)S * 11 + 1;
  CHK(ensure(ctx->st_buf, nd * sizeof(double) + ni * sizeof(int) + 256));
  double* d = as<double>(ctx->st_buf);
  auto take = [&](size_t n) {
    double* r = d;
    d += n;
    return r;
  };
  f->theta = take((size_t)S * NP);
  f->psi = take((size_t)S * NP);
  f->theta_trial = take((size_t)S * NP);
  f->g = take((size_t)S * NP);
  f->p = take((size_t)S * NP);
  f->H = take((size_t)S * NP * NP);
  f->V = take((size_t)S * NP * NP);
  f->g_trial = take((size_t)S * NP);
  f->H_trial = take((size_t)S * NP * NP);
  f->u0 = take((size_t)S * 2);
  f->f = take(S);
  f->f_full = take(S);
  f->f_trial = take(S);
  f->pred = take(S);
  f->delta = take(S);
  f->pnorm = take(S);
  take(S);
  int* ip = reinterpret_cast<int*>(d);
  f->iter = ip;
  f->status = ip + S;
  f->active = ip + 2 * S;
  f->need_full = ip + 3 * S;
  f->n_full = ip + 4 * S;
  f->flags = ip + 5 * S;
  f->samp = ip + 6 * S;
  f->sw = ip + 7 * S;
  f->fa = ip + 8 * S;
  f->fb = ip + 9 * S;
  f->n_acc = ip + 10 * S;
  f->n_active = ip + 11 * S;
  return CELESTE_OK;
}

int check_opts(const celeste_fit_opts* o) {
  if (!o) return fail(CELESTE_E_INVALID, "opts is NULL");
  if (o->max_iter < 1 || o->max_iter > 100000) return fail(CELESTE_E_INVALID, "max_iter must be in 1..100000");
  if (o->init_mode != CELESTE_INIT_AS_GIVEN && o->init_mode != CELESTE_INIT_PLAIN &&
      o->init_mode != CELESTE_INIT_SURROGATE)
    return fail(CELESTE_E_INVALID, "init_mode %d not known", o->init_mode);
  if (!(o->pred_rtol >= 0.0) || !(o->curv_tol >= 0.0) || !(o->delta0 > 0.0) || !(o->delta_max >= o->delta0) ||
      !(o->delta_min >= 0.0) || !(o->eta >= 0.0 && o->eta < 1.0) || !(o->u_box > 0.0))
    return fail(CELESTE_E_INVALID, "fit options out of range");
  return CELESTE_OK;
}

// Enqueues one trust-region iteration over all sources (each kernel skips sources
// whose flag is clear).
// Persistent-grid size of the value+gradient+Hessian kernel for a fit over P: the compute units
// times the chosen blocks per compute unit, or (persistent < 0) times the blocks the launched kernel
// instance keeps resident on one.
int fit_grid(celeste_ctx* ctx, const Packed& P) {
  int bpc = ctx->persistent;
  if (bpc < 0) {
    HIPCHK(eval_full_blocks_per_cu(ctx->block, full_variant(ctx), ctx->tile_log2, P.prof.n_exp, P.prof.n_dev, &bpc));
    bpc = std::max(1, bpc);
  }
  ctx->pgrid = ctx->n_cu * bpc;
  ctx->stats.fit_grid_blocks = ctx->pgrid;
  return CELESTE_OK;
}

// The device work queue of a fit over P's work items (persistent mode).
int fit_queue(celeste_ctx* ctx, const Packed& P, WorkQueue* q) {
  CHK(ensure(ctx->qbuf, sizeof(int) * ((size_t)P.n_items + 64)));
  int* b = as<int>(ctx->qbuf);
  q->hdr = b;
  q->items = b + 64;
  q->srcs = as<SrcDev>(ctx->srcs);
  return CELESTE_OK;
}

int enqueue_iteration(celeste_ctx* ctx, const Packed& P, const FitDev& F, const FitParams& fp, hipStream_t st,
                      PhaseTimer* T, const WorkQueue* Q = nullptr) {
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  const WorkItem* items = as<WorkItem>(ctx->items);
  const SrcDev* srcs = as<SrcDev>(ctx->srcs);
  float* tables = as<float>(ctx->tables);
  double* parts = as<double>(ctx->partials);
  const double* ic = as<double>(ctx->img_const);
  T->mark(0, st);
  if (Q) HIPCHK(launch_build_queue(*Q, P.n_src, F.need_full, st));
  HIPCHK(launch_setup(imgs, P.n_img, F.theta, F.need_full, P.prof, tables, P.tstride, st));
  T->mark(1, st);
  HIPCHK(launch_eval_full(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.need_full, parts,
                          ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st, nullptr, Q, ctx->pgrid));
  T->mark(2, st);
  HIPCHK(launch_reduce_full(srcs, P.n_src, imgs, parts, ic, F.theta, P.prior, F.need_full, F.f_full, F.g, F.H,
                            ctr_full(ctx), st));
  T->mark(3, st);
  HIPCHK(launch_tr_step(F, P.n_src, fp, st));
  T->mark(4, st);
  HIPCHK(launch_setup(imgs, P.n_img, F.theta_trial, F.active, P.prof, tables, P.tstride, st, false));
  T->mark(5, st);
  HIPCHK(launch_eval_value(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.active, parts,
                           ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st));
  T->mark(6, st);
  HIPCHK(launch_reduce_value(srcs, P.n_src, imgs, parts, ic, F.theta_trial, P.prior, F.active, F.f_trial,
                             ctr_value(ctx), st));
  T->mark(7, st);
  HIPCHK(launch_accept(F, P.n_src, fp, st));
  T->mark(8, st);
  return CELESTE_OK;
}

// The value+gradient+Hessian pass at the current point of the sources flagged need_full (with
// trial derivatives: once, before the first iteration).
int enqueue_current_derivs(celeste_ctx* ctx, const Packed& P, const FitDev& F, hipStream_t st, PhaseTimer* T,
                           const WorkQueue* Q) {
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  double* parts = as<double>(ctx->partials);
  T->mark(0, st);
  if (Q) HIPCHK(launch_build_queue(*Q, P.n_src, F.need_full, st));
  HIPCHK(launch_setup(imgs, P.n_img, F.theta, F.need_full, P.prof, as<float>(ctx->tables), P.tstride, st));
  T->mark(1, st);
  HIPCHK(launch_eval_full(as<WorkItem>(ctx->items), P.n_items, imgs, as<float>(ctx->tables), P.tstride,
                          P.prof.n_exp, P.prof.n_dev, F.need_full, parts, ctx->block, full_variant(ctx),
                          ctx->tile_log2, ctx->e_zero, st, nullptr, Q, ctx->pgrid));
  T->mark(2, st);
  HIPCHK(launch_reduce_full(as<SrcDev>(ctx->srcs), P.n_src, imgs, parts, as<double>(ctx->img_const), F.theta,
                            P.prior, F.need_full, F.f_full, F.g, F.H, ctr_full(ctx), st));
  T->mark(3, st);
  return CELESTE_OK;
}

// One trust-region iteration with trial derivatives (section III-B): the subproblem at the current
// point, the ELBO with its gradient and Hessian at the trial point, the ratio test, and an accepted
// step taking over the trial point's gradient and Hessian.
int enqueue_iteration_td(celeste_ctx* ctx, const Packed& P, const FitDev& F, const FitParams& fp, hipStream_t st,
                         PhaseTimer* T, const WorkQueue* Q) {
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  double* parts = as<double>(ctx->partials);
  T->mark(0, st);
  HIPCHK(launch_tr_step(F, P.n_src, fp, st));
  T->mark(1, st);
  if (Q) HIPCHK(launch_build_queue(*Q, P.n_src, F.active, st));
  HIPCHK(launch_setup(imgs, P.n_img, F.theta_trial, F.active, P.prof, as<float>(ctx->tables), P.tstride, st));
  T->mark(2, st);
  HIPCHK(launch_eval_full(as<WorkItem>(ctx->items), P.n_items, imgs, as<float>(ctx->tables), P.tstride,
                          P.prof.n_exp, P.prof.n_dev, F.active, parts, ctx->block, full_variant(ctx),
                          ctx->tile_log2, ctx->e_zero, st, nullptr, Q, ctx->pgrid));
  T->mark(3, st);
  HIPCHK(launch_reduce_full(as<SrcDev>(ctx->srcs), P.n_src, imgs, parts, as<double>(ctx->img_const),
                            F.theta_trial, P.prior, F.active, F.f_trial, F.g_trial, F.H_trial, ctr_trial(ctx), st));
  T->mark(4, st);
  HIPCHK(launch_accept(F, P.n_src, fp, st));
  T->mark(5, st);
  return CELESTE_OK;
}

void accumulate_phases_td(celeste_ctx* ctx, PhaseTimer& T) {
  if (!T.on) return;
  celeste_stats& s = ctx->stats;
  s.ms_tr += T.span(0, 1);
  s.ms_setup += T.span(1, 2);
  s.ms_full += T.span(2, 3);
  s.ms_reduce_full += T.span(3, 4);
  s.ms_accept += T.span(4, 5);
}

void accumulate_phases(celeste_ctx* ctx, PhaseTimer& T) {
  if (!T.on) return;
  celeste_stats& s = ctx->stats;
  s.ms_setup += T.span(0, 1) + T.span(4, 5);
  s.ms_full += T.span(1, 2);
  s.ms_reduce_full += T.span(2, 3);
  s.ms_tr += T.span(3, 4);
  s.ms_value += T.span(5, 6);
  s.ms_reduce_value += T.span(6, 7);
  s.ms_accept += T.span(7, 8);
}

// Host wall clock of the fits' stages (profile mode only): stage k ends at a call; the stream
// is drained first.
struct StageClock {
  bool on;
  std::chrono::steady_clock::time_point t_last = std::chrono::steady_clock::now();
  explicit StageClock(bool on_) : on(on_) {}
  void operator()(double& acc, hipStream_t s) {
    if (!on) return;
    (void)hipStreamSynchronize(s);
    const auto now = std::chrono::steady_clock::now();
    acc += std::chrono::duration<double, std::milli>(now - t_last).count();
    t_last = now;
  }
};

// The common start of the trust-region and L-BFGS fits: validation, packing, metadata upload
// and pixel check, the fit state (F), and the start (plain, surrogate with fallback, or as
// given) with its ELBO in F.f; a source whose start is not finite is not fitted.  th receives
// the host copy of theta_inout.
int fit_begin(celeste_ctx* ctx, const celeste_batch* b, const double* theta_inout, int init_mode,
              const FitParams& fp, hipStream_t st, StageClock& stage, Packed* Pp, FitDev* Fp,
              std::vector<double>* thp) {
  Packed& P = *Pp;
  FitDev& F = *Fp;
  std::vector<double>& th = *thp;
  HIPCHK(hipSetDevice(ctx->device));
  const int S = P.n_src;
  th.resize(NP * (size_t)S);
  if (b->mem_kind == CELESTE_MEM_HOST)
    std::memcpy(th.data(), theta_inout, sizeof(double) * th.size());
  else {
    HIPCHK(hipMemcpyAsync(th.data(), theta_inout, sizeof(double) * th.size(), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
  }
  if (init_mode == CELESTE_INIT_SURROGATE && !ctx->net)
    return fail(CELESTE_E_INVALID, "CELESTE_INIT_SURROGATE needs a network (celeste_ctx_set_surrogate)");
  for (int s = 0; s < S; ++s) {
    if (init_mode != CELESTE_INIT_AS_GIVEN) {
      if (!finite(th[(size_t)s * NP]) || !finite(th[(size_t)s * NP + 1]))
        return fail(CELESTE_E_INVALID, "theta[%d]: position must be finite", s);
    } else {
      CHK(check_theta(th.data() + (size_t)s * NP, s));
    }
  }
  stage(ctx->stats.ms_host_pack, st);
  CHK(prepare(ctx, b, &P, st));
  stage(ctx->stats.ms_prepare, st);
  CHK(alloc_fit(ctx, S, &F));
  HIPCHK(hipMemcpyAsync(F.theta, th.data(), sizeof(double) * th.size(), hipMemcpyHostToDevice, st));
  HIPCHK(launch_zero_int(F.flags, S, st));
  const ImgDev* imgs0 = as<ImgDev>(ctx->imgs);
  if (init_mode == CELESTE_INIT_SURROGATE) {
    // network start (from the catalog positions in F.theta) into theta_trial, plain start into theta,
    // both evaluated; the better one is kept
    CHK(ensure(ctx->sur, sizeof(float) * NP * (size_t)S));
    CHK(surrogate_predict(ctx->net, as<SrcDev>(ctx->srcs), S, imgs0, F.theta, as<float>(ctx->sur), st));
    HIPCHK(launch_psi_to_theta(as<float>(ctx->sur), F.theta, F.theta_trial, S, fp.u_box, st));
    stage(ctx->stats.ms_net, st);
    HIPCHK(launch_plain_init(as<SrcDev>(ctx->srcs), S, imgs0, P.prior, F.theta, st));
    for (int k = 0; k < 2; ++k) {
      double* tk = k == 0 ? F.theta : F.theta_trial;
      HIPCHK(launch_setup(imgs0, P.n_img, tk, nullptr, P.prof, as<float>(ctx->tables), P.tstride, st, false));
      HIPCHK(launch_eval_value(as<WorkItem>(ctx->items), P.n_items, imgs0, as<float>(ctx->tables), P.tstride,
                               P.prof.n_exp, P.prof.n_dev, nullptr, as<double>(ctx->partials), ctx->vblock, ctx->variant,
                             ctx->vtile_log2, ctx->e_zero, st));
      HIPCHK(launch_reduce_value(as<SrcDev>(ctx->srcs), S, imgs0, as<double>(ctx->partials),
                                 as<double>(ctx->img_const), tk, P.prior, nullptr, k == 0 ? F.f : F.f_trial,
                                 ctr_value(ctx), st));
      ctx->stats.value_launches += 1;
    }
    HIPCHK(launch_choose_start(F, S, st));
  } else if (init_mode == CELESTE_INIT_PLAIN) {
    HIPCHK(launch_plain_init(as<SrcDev>(ctx->srcs), S, imgs0, P.prior, F.theta, st));
  }
  HIPCHK(launch_fit_init(F, S, fp, st));
  if (init_mode != CELESTE_INIT_SURROGATE) {
    // the start's ELBO (the surrogate path has it from choosing between the two starts: both lie
    // inside the boxes, where the transform round trip of the fit set-up moves a parameter by
    // rounding, or by at most 1e-9 of its box where a start sits on the box edge)
    const ImgDev* imgs = as<ImgDev>(ctx->imgs);
    HIPCHK(launch_setup(imgs, P.n_img, F.theta, nullptr, P.prof, as<float>(ctx->tables), P.tstride, st, false));
    HIPCHK(launch_eval_value(as<WorkItem>(ctx->items), P.n_items, imgs, as<float>(ctx->tables), P.tstride,
                             P.prof.n_exp, P.prof.n_dev, nullptr, as<double>(ctx->partials), ctx->vblock,
                             ctx->variant, ctx->vtile_log2, ctx->e_zero, st));
    HIPCHK(launch_reduce_value(as<SrcDev>(ctx->srcs), S, imgs, as<double>(ctx->partials),
                               as<double>(ctx->img_const), F.theta, P.prior, nullptr, F.f, ctr_value(ctx), st));
    ctx->stats.value_launches += 1;
  }
  HIPCHK(launch_fit_start(F, S, st));
  return CELESTE_OK;
}

// Per-source results of a fit from its device state; theta_inout receives the parameters.
int fit_results(celeste_ctx* ctx, const celeste_batch* b, const FitDev& F, int S, std::vector<double>& th,
                double* theta_inout, celeste_fit_result* res, hipStream_t st, StageClock& stage) {
  std::vector<double> fv(S), pred(S), delta(S);
  std::vector<int> iter(S), status(S), nfull(S), flags(S), nacc(S);
  HIPCHK(hipMemcpyAsync(th.data(), F.theta, sizeof(double) * th.size(), hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(fv.data(), F.f, sizeof(double) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(pred.data(), F.pred, sizeof(double) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(delta.data(), F.delta, sizeof(double) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(iter.data(), F.iter, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(status.data(), F.status, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(nfull.data(), F.n_full, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(flags.data(), F.flags, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(nacc.data(), F.n_acc, sizeof(int) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  if (b->mem_kind == CELESTE_MEM_HOST)
    std::memcpy(theta_inout, th.data(), sizeof(double) * th.size());
  else {
    HIPCHK(hipMemcpyAsync(theta_inout, F.theta, sizeof(double) * th.size(), hipMemcpyDeviceToDevice, st));
    HIPCHK(hipStreamSynchronize(st));
  }
  stage(ctx->stats.ms_results, st);
  for (int s = 0; s < S; ++s) {
    res[s].elbo = fv[s];
    res[s].pred_gain = pred[s];
    res[s].delta = delta[s];
    res[s].iters = iter[s];
    res[s].status = status[s];
    res[s].n_full_evals = nfull[s];
    res[s].n_accepted = nacc[s];
    res[s].reserved = 0;
    res[s].flags = flags[s];
  }
  return CELESTE_OK;
}

// Replays (graph) or enqueues (eager) `iteration` until no source is active or max_loops loop
// steps; the host reads the device's active count of every `poll` steps.
// count(stats) records the launches of one step (replayed or enqueued) up to the poll that ends the loop.
template <class Iter, class Count>
int run_loop(celeste_ctx* ctx, hipStream_t st, int max_loops, int poll, bool use_graph, const int* n_active_dev,
             PhaseTimer& T, Iter iteration, Count count, void (*account)(celeste_ctx*, PhaseTimer&)) {
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  if (use_graph) {
    PhaseTimer none;
    HIPCHK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
    int rc = iteration(&none);
    hipError_t e2 = hipStreamEndCapture(st, &graph);
    if (rc != CELESTE_OK) {
      if (graph) (void)hipGraphDestroy(graph);
      return rc;
    }
    HIPCHK(e2);
    HIPCHK(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
  }
  // The count is read one poll behind the launches, so that the device always has iterations to run: reading it
  // before the next launch left the device idle for 40 us an iteration of a single source's fit (of 185).
  // The iterations launched past the one that left nothing active find every source inactive.  With phase
  // times (T.on, one iteration's events) each iteration is waited for.
  int rc = ensure_host(ctx->h_poll, 2 * sizeof(int));
  volatile int* slot = as<int>(ctx->h_poll);
  hipEvent_t ev[2] = {};
  for (auto& e : ev)
    if (rc == CELESTE_OK && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess)
      rc = fail(CELESTE_E_DEVICE, "event creation failed");
  int polls = 0, since = 0, covered[2] = {};
  bool active = true;
  const auto read_poll = [&](int k) {   // waits for poll k; its iterations are counted
    const hipError_t e = hipEventSynchronize(ev[k & 1]);
    if (e != hipSuccess) {
      rc = fail(CELESTE_E_DEVICE, "active-count readback: %s", hipGetErrorString(e));
      return;
    }
    for (int i = 0; i < covered[k & 1]; ++i) {
      ctx->stats.iterations += 1;
      count(ctx->stats);
    }
    account(ctx, T);
    active = slot[k & 1] > 0;
  };
  for (int it = 0; it < max_loops && active && rc == CELESTE_OK; ++it) {
    if (exec) {
      hipError_t e = hipGraphLaunch(exec, st);
      if (e != hipSuccess) {
        rc = fail(CELESTE_E_DEVICE, "hipGraphLaunch: %s", hipGetErrorString(e));
        break;
      }
    } else {
      rc = iteration(&T);
      if (rc != CELESTE_OK) break;
    }
    ++since;
    if ((it + 1) % poll != 0 && it + 1 != max_loops) continue;
    hipError_t e = hipMemcpyAsync(const_cast<int*>(slot) + (polls & 1), n_active_dev, sizeof(int), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipEventRecord(ev[polls & 1], st);
    if (e != hipSuccess) {
      rc = fail(CELESTE_E_DEVICE, "active-count readback: %s", hipGetErrorString(e));
      break;
    }
    covered[polls & 1] = since;
    since = 0;
    ++polls;
    const bool last = it + 1 == max_loops;
    if (polls > 1 && !T.on) read_poll(polls - 2);
    if (rc == CELESTE_OK && active && (last || T.on)) read_poll(polls - 1);
  }
  for (auto& e : ev)
    if (e) (void)hipEventDestroy(e);
  if (exec) {   // not while a launch of it runs
    (void)hipStreamSynchronize(st);
    (void)hipGraphExecDestroy(exec);
  }
  if (graph) (void)hipGraphDestroy(graph);
  return rc;
}

int run_fit(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_fit_opts* o,
            celeste_fit_result* res, hipStream_t st, bool batched, double* start_elbo = nullptr,
            bool start_only = false) {
  StageClock stage(ctx->profile != 0);
  Packed P;
  CHK(validate_and_pack(ctx, b, &P));
  if (start_only) {
    if (!o) return fail(CELESTE_E_INVALID, "opts is NULL");
    celeste_fit_opts o2 = *o;
    o2.max_iter = 1;
    CHK(check_opts(&o2));
  } else {
    CHK(check_opts(o));
  }
  if (!theta_inout || (!res && !start_only)) return fail(CELESTE_E_INVALID, "theta_inout and results must not be NULL");
  const int S = P.n_src;
  FitParams fp{};
  fp.max_iter = o->max_iter;
  fp.pred_rtol = o->pred_rtol;
  fp.curv_tol = o->curv_tol;
  fp.delta0 = o->delta0;
  fp.delta_max = o->delta_max;
  fp.delta_min = o->delta_min;
  fp.eta = o->eta;
  fp.u_box = o->u_box;
  fp.tr_chol = ctx->tr_chol;
  fp.trial_derivs = ctx->trial_derivs;
  fp.tr_ctr = as<unsigned long long>(ctx->ctr) + 3;
  FitDev F;
  std::vector<double> th;
  CHK(fit_begin(ctx, b, theta_inout, o->init_mode, fp, st, stage, &P, &F, &th));
  // the batch's per-source metadata exists from here on (fit_begin's upload may reallocate it)
  fp.srcs = as<SrcDev>(ctx->srcs);
  fp.taken_px = ctr_taken(ctx);
  if (start_only) {
    if (b->mem_kind == CELESTE_MEM_HOST) {
      HIPCHK(hipMemcpyAsync(theta_inout, F.theta, sizeof(double) * th.size(), hipMemcpyDeviceToHost, st));
      if (start_elbo) HIPCHK(hipMemcpyAsync(start_elbo, F.f, sizeof(double) * S, hipMemcpyDeviceToHost, st));
    } else {
      HIPCHK(hipMemcpyAsync(theta_inout, F.theta, sizeof(double) * th.size(), hipMemcpyDeviceToDevice, st));
      if (start_elbo) HIPCHK(hipMemcpyAsync(start_elbo, F.f, sizeof(double) * S, hipMemcpyDeviceToDevice, st));
    }
    HIPCHK(hipStreamSynchronize(st));
    return CELESTE_OK;
  }
  stage(ctx->stats.ms_start, st);
  PhaseTimer T;
  CHK(T.init(ctx->profile != 0));
  const int poll = (batched && !T.on) ? std::max(1, o->poll_every) : 1;
  const bool graph = batched && ctx->use_graph && !T.on;
  WorkQueue Q;
  ctx->stats.fit_grid_blocks = 0;
  if (ctx->persistent) {
    CHK(fit_queue(ctx, P, &Q));
    CHK(fit_grid(ctx, P));
  }
  // items that all run at once need no list to be drawn from (its launch: 4.6 us an iteration)
  const WorkQueue* Qp = ctx->persistent && P.n_items > ctx->pgrid ? &Q : nullptr;
  if (fp.trial_derivs) {
    // the start's gradient and Hessian, then iterations that evaluate them at every trial point
    CHK(enqueue_current_derivs(ctx, P, F, st, &T, Qp));
    ctx->stats.full_launches += 1;
    if (T.on) {
      HIPCHK(hipStreamSynchronize(st));
      ctx->stats.ms_setup += T.span(0, 1);
      ctx->stats.ms_full += T.span(1, 2);
      ctx->stats.ms_reduce_full += T.span(2, 3);
    }
    CHK(run_loop(ctx, st, o->max_iter + 1, poll, graph, F.n_active, T,
                 [&](PhaseTimer* t) { return enqueue_iteration_td(ctx, P, F, fp, st, t, Qp); },
                 [](celeste_stats& c) { c.full_launches += 1; }, accumulate_phases_td));
  } else {
    CHK(run_loop(ctx, st, o->max_iter + 1, poll, graph, F.n_active, T,
                 [&](PhaseTimer* t) { return enqueue_iteration(ctx, P, F, fp, st, t, Qp); },
                 [](celeste_stats& c) {
                   c.full_launches += 1;
                   c.value_launches += 1;
                 },
                 accumulate_phases));
  }
  stage(ctx->stats.ms_loop, st);
  return fit_results(ctx, b, F, S, th, theta_inout, res, st, stage);
}

// Trust-region fit whose early phase fits a pixel-subsampled estimate of the ELBO (8-row
// blocks kept by `keep`, weighted 1 / keep_prob): each source moves to the full ELBO when its
// model's predicted gain on the estimate falls to switch_rtol max(1, |L|), and then runs the
// fit's own stopping rule.  One iteration evaluates, per source, on whichever objective it is in.
int run_fit_sampled(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_fit_opts* o,
                    const uint8_t* keep, const int64_t* keep_off, double keep_prob, double switch_rtol,
                    celeste_fit_result* res, hipStream_t st) {
  StageClock stage(ctx->profile != 0);
  if (!keep || !keep_off) return fail(CELESTE_E_INVALID, "keep and keep_off must not be NULL");
  if (!(keep_prob > 0.0 && keep_prob <= 1.0)) return fail(CELESTE_E_INVALID, "keep_prob must be in (0, 1]");
  if (!(switch_rtol > 0.0)) return fail(CELESTE_E_INVALID, "switch_rtol must be > 0");
  Packed P;
  CHK(validate_and_pack(ctx, b, &P));
  CHK(check_opts(o));
  if (!theta_inout || !res) return fail(CELESTE_E_INVALID, "theta_inout and results must not be NULL");
  if (keep_off[0] != 0) return fail(CELESTE_E_INVALID, "keep_off[0] must be 0");
  for (int i = 0; i < P.n_img; ++i)
    if (keep_off[i + 1] - keep_off[i] != (b->images[i].h + 7) / 8)
      return fail(CELESTE_E_INVALID, "image %d: keep_off must give (h + 7) / 8 blocks", i);
  const int S = P.n_src;
  FitParams fp{};
  fp.max_iter = o->max_iter;
  fp.pred_rtol = o->pred_rtol;
  fp.curv_tol = o->curv_tol;
  fp.delta0 = o->delta0;
  fp.delta_max = o->delta_max;
  fp.delta_min = o->delta_min;
  fp.eta = o->eta;
  fp.u_box = o->u_box;
  fp.switch_rtol = switch_rtol;
  fp.tr_chol = ctx->tr_chol;
  fp.tr_ctr = as<unsigned long long>(ctx->ctr) + 3;
  FitDev F;
  std::vector<double> th;
  CHK(fit_begin(ctx, b, theta_inout, o->init_mode, fp, st, stage, &P, &F, &th));
  // the subsampled pack: the dense image records (pixels already staged) with work items over
  // the kept blocks only
  std::vector<ImgDev> img_copy(P.imgs, P.imgs + P.n_img);
  std::vector<SrcDev> src_copy(P.srcs, P.srcs + P.n_src);
  Packed Ps = P;
  Ps.imgs = img_copy.data();
  Ps.srcs = src_copy.data();
  CHK(subsample_items(ctx, b, &Ps, keep, keep_off));
  CHK(ensure(ctx->imgs_s, sizeof(ImgDev) * Ps.n_img));
  CHK(ensure(ctx->items_s, Ps.items_bytes));
  CHK(ensure(ctx->srcs_s, sizeof(SrcDev) * Ps.n_src));
  CHK(ensure(ctx->partials_s, sizeof(double) * (size_t)NACC * std::max(1, Ps.n_items)));
  HIPCHK(hipMemcpyAsync(ctx->imgs_s.p, Ps.imgs, sizeof(ImgDev) * Ps.n_img, hipMemcpyHostToDevice, st));
  if (Ps.n_items > 0)
    HIPCHK(hipMemcpyAsync(ctx->items_s.p, Ps.items, Ps.items_bytes, hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(ctx->srcs_s.p, Ps.srcs, sizeof(SrcDev) * Ps.n_src, hipMemcpyHostToDevice, st));
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  const WorkItem* items = as<WorkItem>(ctx->items);
  const SrcDev* srcs = as<SrcDev>(ctx->srcs);
  const ImgDev* imgs_s = as<ImgDev>(ctx->imgs_s);
  const WorkItem* items_s = as<WorkItem>(ctx->items_s);
  const SrcDev* srcs_s = as<SrcDev>(ctx->srcs_s);
  const int* kept = reinterpret_cast<int*>(as<unsigned char>(ctx->items_s) + Ps.o_kept);
  float* tables = as<float>(ctx->tables);
  double* parts = as<double>(ctx->partials);
  double* parts_s = as<double>(ctx->partials_s);
  const double* ic = as<double>(ctx->img_const);
  const double w = 1.0 / keep_prob;
  // every fitted source starts on the subsampled objective: its value there at the start
  HIPCHK(launch_fill_int(F.samp, S, 1, st));
  HIPCHK(launch_split(F.active, F.samp, F.fa, F.fb, S, st));
  HIPCHK(launch_setup(imgs, P.n_img, F.theta, F.fb, P.prof, tables, P.tstride, st, false));
  HIPCHK(launch_eval_value(items_s, Ps.n_items, imgs_s, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.fb, parts_s,
                           ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st, kept));
  HIPCHK(launch_reduce_value(srcs_s, S, imgs_s, parts_s, ic, F.theta, P.prior, F.fb, F.f, ctr_value(ctx), st, w));
  stage(ctx->stats.ms_start, st);
  PhaseTimer T;
  CHK(T.init(ctx->profile != 0));
  auto iteration = [&](PhaseTimer* t) -> int {
    t->mark(0, st);
    HIPCHK(launch_split(F.need_full, F.samp, F.fa, F.fb, S, st));
    HIPCHK(launch_setup(imgs, P.n_img, F.theta, F.need_full, P.prof, tables, P.tstride, st));
    t->mark(1, st);
    HIPCHK(launch_eval_full(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.fa, parts,
                            ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st));
    HIPCHK(launch_eval_full(items_s, Ps.n_items, imgs_s, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.fb, parts_s,
                            ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st, kept));
    t->mark(2, st);
    HIPCHK(launch_reduce_full(srcs, S, imgs, parts, ic, F.theta, P.prior, F.fa, F.f_full, F.g, F.H, ctr_full(ctx), st));
    HIPCHK(launch_reduce_full(srcs_s, S, imgs_s, parts_s, ic, F.theta, P.prior, F.fb, F.f_full, F.g, F.H,
                              ctr_full(ctx), st, w));
    t->mark(3, st);
    HIPCHK(launch_tr_step(F, S, fp, st));
    t->mark(4, st);
    HIPCHK(launch_split(F.active, F.samp, F.fa, F.fb, S, st));
    HIPCHK(launch_setup(imgs, P.n_img, F.theta_trial, F.active, P.prof, tables, P.tstride, st, false));
    t->mark(5, st);
    HIPCHK(launch_eval_value(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.fa, parts,
                             ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st));
    HIPCHK(launch_eval_value(items_s, Ps.n_items, imgs_s, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.fb, parts_s,
                             ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st, kept));
    t->mark(6, st);
    HIPCHK(launch_reduce_value(srcs, S, imgs, parts, ic, F.theta_trial, P.prior, F.fa, F.f_trial, ctr_value(ctx), st));
    HIPCHK(launch_reduce_value(srcs_s, S, imgs_s, parts_s, ic, F.theta_trial, P.prior, F.fb, F.f_trial,
                               ctr_value(ctx), st, w));
    t->mark(7, st);
    HIPCHK(launch_accept(F, S, fp, st));
    t->mark(8, st);
    return CELESTE_OK;
  };
  const int poll = T.on ? 1 : std::max(1, o->poll_every);
  // the switches are loop steps that are not iterations: room for one per source
  CHK(run_loop(ctx, st, o->max_iter + 2, poll, ctx->use_graph && !T.on, F.n_active, T, iteration,
               [](celeste_stats& c) {
                 c.full_launches += 1;
                 c.value_launches += 1;
               },
               accumulate_phases));
  stage(ctx->stats.ms_loop, st);
  return fit_results(ctx, b, F, S, th, theta_inout, res, st, stage);
}

int check_lbfgs_opts(const celeste_lbfgs_opts* o) {
  if (!o) return fail(CELESTE_E_INVALID, "opts is NULL");
  if (o->max_iter < 1 || o->max_iter > 1000000) return fail(CELESTE_E_INVALID, "max_iter must be in 1..1e6");
  if (o->memory < 1 || o->memory > LBFGS_MAX_MEMORY) return fail(CELESTE_E_INVALID, "memory must be in 1..32");
  if (o->max_backtracks < 1 || o->max_backtracks > 60) return fail(CELESTE_E_INVALID, "max_backtracks must be in 1..60");
  if (o->init_mode != CELESTE_INIT_AS_GIVEN && o->init_mode != CELESTE_INIT_PLAIN &&
      o->init_mode != CELESTE_INIT_SURROGATE)
    return fail(CELESTE_E_INVALID, "unknown init_mode %d", o->init_mode);
  if (o->max_loops < 0) return fail(CELESTE_E_INVALID, "max_loops must be >= 0");
  if (!(o->pred_rtol > 0.0) || !(o->armijo_c1 > 0.0 && o->armijo_c1 < 0.5) || !(o->u_box > 0.0))
    return fail(CELESTE_E_INVALID, "pred_rtol and u_box must be > 0 and armijo_c1 in (0, 1/2)");
  return CELESTE_OK;
}

void accumulate_lbfgs_phases(celeste_ctx* ctx, PhaseTimer& T) {
  if (!T.on) return;
  celeste_stats& s = ctx->stats;
  s.ms_setup += T.span(0, 1) + T.span(4, 5);
  s.ms_grad += T.span(1, 2);
  s.ms_reduce_grad += T.span(2, 3);
  s.ms_lbfgs += T.span(3, 4) + T.span(7, 8);
  s.ms_value += T.span(5, 6);
  s.ms_reduce_value += T.span(6, 7);
}

int run_lbfgs(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_lbfgs_opts* o,
              celeste_fit_result* res, hipStream_t st) {
  StageClock stage(ctx->profile != 0);
  Packed P;
  CHK(validate_and_pack(ctx, b, &P));
  CHK(check_lbfgs_opts(o));
  if (!theta_inout || !res) return fail(CELESTE_E_INVALID, "theta_inout and results must not be NULL");
  const int S = P.n_src;
  FitParams fp{};
  fp.max_iter = o->max_iter;
  fp.delta0 = 1.0;
  fp.u_box = o->u_box;
  FitDev F;
  std::vector<double> th;
  CHK(fit_begin(ctx, b, theta_inout, o->init_mode, fp, st, stage, &P, &F, &th));
  // L-BFGS state: pairs, rho, gradients and scalars, then the integer counters
  const int m = o->memory;
  const size_t nd = (size_t)S * (2 * (size_t)m * NP + m + NP + 1);
  const size_t ni = (size_t)S * 5;
  CHK(ensure(ctx->lb_buf, nd * sizeof(double) + ni * sizeof(int) + 256));
  LbfgsDev X;
  {
    double* d = as<double>(ctx->lb_buf);
    auto take = [&d](size_t n) {
      double* r = d;
      d += n;
      return r;
    };
    X.S = take((size_t)S * m * NP);
    X.Y = take((size_t)S * m * NP);
    X.rho = take((size_t)S * m);
    X.gpsi = take((size_t)S * NP);
    X.gp = take(S);
    int* ip = reinterpret_cast<int*>(d);
    X.n_pairs = ip;
    X.head = ip + S;
    X.ls = ip + 2 * S;
    X.n_val = ip + 3 * S;
    X.in_ls = ip + 4 * S;
  }
  LbfgsParams lp;
  lp.max_iter = o->max_iter;
  lp.memory = m;
  lp.max_backtracks = o->max_backtracks;
  lp.pred_rtol = o->pred_rtol;
  lp.c1 = o->armijo_c1;
  lp.u_box = o->u_box;
  HIPCHK(launch_lbfgs_init(X, S, st));
  stage(ctx->stats.ms_start, st);
  PhaseTimer T;
  CHK(T.init(ctx->profile != 0));
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  const WorkItem* items = as<WorkItem>(ctx->items);
  const SrcDev* srcs = as<SrcDev>(ctx->srcs);
  float* tables = as<float>(ctx->tables);
  double* parts = as<double>(ctx->partials);
  const double* ic = as<double>(ctx->img_const);
  auto iteration = [&](PhaseTimer* t) -> int {
    t->mark(0, st);
    HIPCHK(launch_setup(imgs, P.n_img, F.theta, F.need_full, P.prof, tables, P.tstride, st));
    t->mark(1, st);
    HIPCHK(launch_eval_grad(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, F.need_full,
                            parts, ctx->block, full_variant(ctx), ctx->tile_log2, ctx->e_zero, st));
    t->mark(2, st);
    HIPCHK(launch_reduce_grad(srcs, P.n_src, imgs, parts, ic, F.theta, P.prior, F.need_full, F.f_full, F.g,
                              ctr_grad(ctx), st));
    t->mark(3, st);
    HIPCHK(launch_zero_int(F.n_active, 1, st));
    HIPCHK(launch_lbfgs_dir(F, X, P.n_src, lp, st));
    t->mark(4, st);
    HIPCHK(launch_setup(imgs, P.n_img, F.theta_trial, X.in_ls, P.prof, tables, P.tstride, st, false));
    t->mark(5, st);
    HIPCHK(launch_eval_value(items, P.n_items, imgs, tables, P.tstride, P.prof.n_exp, P.prof.n_dev, X.in_ls, parts,
                             ctx->vblock, ctx->variant, ctx->vtile_log2, ctx->e_zero, st));
    t->mark(6, st);
    HIPCHK(launch_reduce_value(srcs, P.n_src, imgs, parts, ic, F.theta_trial, P.prior, X.in_ls, F.f_trial,
                               ctr_value(ctx), st));
    t->mark(7, st);
    HIPCHK(launch_lbfgs_accept(F, X, P.n_src, lp, st));
    t->mark(8, st);
    return CELESTE_OK;
  };
  const int max_loops = o->max_loops > 0 ? o->max_loops : 4 * o->max_iter + 64;
  const int poll = T.on ? 1 : std::max(1, o->poll_every);
  CHK(run_loop(ctx, st, max_loops, poll, ctx->use_graph && !T.on, F.n_active, T, iteration,
               [](celeste_stats& c) {
                 c.grad_launches += 1;
                 c.value_launches += 1;
               },
               accumulate_lbfgs_phases));
  stage(ctx->stats.ms_loop, st);
  return fit_results(ctx, b, F, S, th, theta_inout, res, st, stage);
}

}  // namespace

extern "C" {

int celeste_newton_fit(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_fit_opts* opts,
                       celeste_fit_result* result) {
  if (!b) return fail(CELESTE_E_INVALID, "batch is NULL");
  if (b->n_sources != 1) return fail(CELESTE_E_INVALID, "celeste_newton_fit takes exactly one source");
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  return run_fit(ctx, b, theta_inout, opts, result, ctx->stream, false);
}

int celeste_batch_fit(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_fit_opts* opts,
                      celeste_fit_result* results, void* stream) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  return run_fit(ctx, b, theta_inout, opts, results, pick(ctx, stream), true);
}

int celeste_batch_fit_sampled(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout,
                              const celeste_fit_opts* opts, const uint8_t* keep, const int64_t* keep_off,
                              double keep_prob, double switch_rtol, celeste_fit_result* results, void* stream) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  return run_fit_sampled(ctx, b, theta_inout, opts, keep, keep_off, keep_prob, switch_rtol, results,
                         pick(ctx, stream));
}

void celeste_lbfgs_opts_default(celeste_lbfgs_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->max_iter = 1000;
  o->memory = 10;
  o->max_backtracks = 30;
  o->init_mode = CELESTE_INIT_PLAIN;
  o->poll_every = 4;
  o->max_loops = 0;
  o->pred_rtol = 1e-8;
  o->armijo_c1 = 1e-4;
  o->u_box = 3.0;
}

int celeste_lbfgs_fit(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_lbfgs_opts* opts,
                      celeste_fit_result* results, void* stream) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  return run_lbfgs(ctx, b, theta_inout, opts, results, pick(ctx, stream));
}

}  // extern "C"

// =============================================================================== surrogate glue

namespace {

struct HostBox {
  double lo, hi;
  int kind;   // 0 identity, 1 scaled logistic, 2 exp
};

HostBox host_box(int i, const double* u0, double u_box) {
  if (i == 0 || i == 1) return {u0[i] - u_box, u0[i] + u_box, 1};
  if (i == 2 || i == 3) return {1e-4, 1.0 - 1e-4, 1};
  if (i == 4) return {0.01, 0.99, 1};
  if (i == 6) return {0.2, 15.0, 1};
  if (i == 9 || i == 10 || i >= 19) return {0.0, 0.0, 2};
  return {0.0, 0.0, 0};
}

}  // namespace

extern "C" {

int celeste_ctx_set_surrogate(celeste_ctx* ctx, celeste_net* net) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  ctx->net = net;
  return CELESTE_OK;
}

int celeste_make_patches(celeste_ctx* ctx, const celeste_batch* b, const double* theta, void* out) {
  Packed P;
  CHK(validate_and_pack(ctx, b, &P, nullptr, Pack::kNoItems));
  if (!theta || !out) return fail(CELESTE_E_INVALID, "theta and out must not be NULL");
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  const double* th = theta;
  if (b->mem_kind == CELESTE_MEM_HOST) {
    CHK(ensure(ctx->theta, sizeof(double) * NP * P.n_src));
    HIPCHK(hipMemcpyAsync(ctx->theta.p, theta, sizeof(double) * NP * P.n_src, hipMemcpyHostToDevice, st));
    th = as<double>(ctx->theta);
  }
  CHK(prepare(ctx, b, &P, st));
  HIPCHK(launch_patches(as<SrcDev>(ctx->srcs), P.n_src, as<ImgDev>(ctx->imgs), th, out, st));
  HIPCHK(hipStreamSynchronize(st));
  return CELESTE_OK;
}

int celeste_theta_to_psi(const double* theta, const double* u0, int64_t n, double u_box, double* psi) {
  if (!theta || !u0 || !psi || n < 0 || !(u_box > 0.0)) return fail(CELESTE_E_INVALID, "bad argument");
  for (int64_t s = 0; s < n; ++s)
    for (int i = 0; i < NP; ++i) {
      const HostBox bx = host_box(i, u0 + 2 * s, u_box);
      const double t = theta[s * NP + i];
      double v = t;
      if (bx.kind == 2) {
        v = std::log(t);
      } else if (bx.kind == 1) {
        const double span = bx.hi - bx.lo;
        const double x = std::min(std::max(t, bx.lo + 1e-9 * span), bx.hi - 1e-9 * span);
        const double f = (x - bx.lo) / span;
        v = std::log(f) - std::log1p(-f);
      }
      psi[s * NP + i] = v;
    }
  return CELESTE_OK;
}

int celeste_psi_to_theta(const double* psi, const double* u0, int64_t n, double u_box, double* theta) {
  if (!theta || !u0 || !psi || n < 0 || !(u_box > 0.0)) return fail(CELESTE_E_INVALID, "bad argument");
  for (int64_t s = 0; s < n; ++s)
    for (int i = 0; i < NP; ++i) {
      const HostBox bx = host_box(i, u0 + 2 * s, u_box);
      const double p = psi[s * NP + i];
      double v = p;
      if (bx.kind == 2) v = std::exp(p);
      else if (bx.kind == 1) v = bx.lo + (bx.hi - bx.lo) / (1.0 + std::exp(-p));
      theta[s * NP + i] = v;
    }
  return CELESTE_OK;
}

}  // extern "C"

// =============================================================================== crowded fields

namespace {

// Bounding boxes [x0, x1) x [y0, y1) of each source's patches (union over its images, in
// image-frame coordinates), for the colouring.
struct Box {
  int64_t x0, x1, y0, y1;
};
constexpr int64_t CELL = 128;   // grid cell of the colouring (>= the usual patch side)

bool overlap(const Box& a, const Box& b) { return a.x0 < b.x1 && b.x0 < a.x1 && a.y0 < b.y1 && b.y0 < a.y1; }

int64_t cell_key(int64_t cx, int64_t cy) { return (cx << 32) ^ (cy & 0xffffffffLL); }

int source_boxes(const celeste_batch* b, std::vector<Box>* out) {
  const int S = b->n_sources;
  if (b->image_offsets[0] != 0) return fail(CELESTE_E_INVALID, "image_offsets[0] must be 0");
  out->resize(S);
  for (int s = 0; s < S; ++s) {
    if (b->image_offsets[s + 1] <= b->image_offsets[s]) return fail(CELESTE_E_INVALID, "source %d has no images", s);
    Box bx{INT64_MAX, INT64_MIN, INT64_MAX, INT64_MIN};
    for (int64_t i = b->image_offsets[s]; i < b->image_offsets[s + 1]; ++i) {
      const celeste_image& im = b->images[i];
      const double ox = im.origin[0], oy = im.origin[1];
      if (!std::isfinite(ox) || !std::isfinite(oy) || std::fabs(ox) > 1e9 || std::fabs(oy) > 1e9 || im.h < 1 ||
          im.w < 1)
        return fail(CELESTE_E_INVALID, "image %lld: bad origin or shape", (long long)i);
      // non-negative cell coordinates: shift by 2^31 before the grid division
      const int64_t x0 = (int64_t)std::floor(ox) + ((int64_t)1 << 31), y0 = (int64_t)std::floor(oy) + ((int64_t)1 << 31);
      bx.x0 = std::min(bx.x0, x0);
      bx.y0 = std::min(bx.y0, y0);
      bx.x1 = std::max(bx.x1, x0 + im.w + (ox != std::floor(ox) ? 1 : 0));
      bx.y1 = std::max(bx.y1, y0 + im.h + (oy != std::floor(oy) ? 1 : 0));
    }
    (*out)[s] = bx;
  }
  return CELESTE_OK;
}

// An image's patch in its field.
struct Patch {
  int field, x, y, w, h;
};

// No two images of the batch on the same field may overlap (single writer per field pixel).  The fields are shared
// out over host threads; each files its patches in a grid of CELL-sided cells, in image order, a chain per cell.
int check_disjoint(const std::vector<Patch>& pt, int n_fields) {
  const int64_t n = (int64_t)pt.size();
  struct Hit {
    int64_t i = INT64_MAX, j = 0;
  };
  Hit hit[TEAM_MAX];
  try {
    team(std::min(team_size(n, 35), n_fields), [&](int t, int nt, Barrier&) {
      const int f0 = (int)((int64_t)n_fields * t / nt), f1 = (int)((int64_t)n_fields * (t + 1) / nt);
      struct Node {
        int img, next;
      };
      std::vector<Node> nodes;
      std::unordered_map<int64_t, int> last;   // newest node of a cell
      last.reserve((size_t)(4 * n / nt));
      for (int64_t i = 0; i < n && hit[t].i == INT64_MAX; ++i) {
        const Patch& a = pt[i];
        if (a.field < f0 || a.field >= f1) continue;
        const int64_t fkey = (int64_t)a.field << 40;
        for (int64_t cy = a.y / CELL; cy <= (a.y + a.h - 1) / CELL; ++cy)
          for (int64_t cx = a.x / CELL; cx <= (a.x + a.w - 1) / CELL && hit[t].i == INT64_MAX; ++cx) {
            auto e = last.emplace(fkey ^ (cx << 20) ^ cy, -1).first;
            for (int k = e->second; k >= 0; k = nodes[k].next) {   // newest first: the last match is the first image
              const Patch& c = pt[nodes[k].img];
              if (c.field == a.field && a.x < c.x + c.w && c.x < a.x + a.w && a.y < c.y + c.h && c.y < a.y + a.h)
                hit[t] = Hit{i, nodes[k].img};
            }
            nodes.push_back(Node{(int)i, e->second});
            e->second = (int)nodes.size() - 1;
          }
      }
    });
  } catch (const std::bad_alloc&) {
    return fail(CELESTE_E_NOMEM, "host allocation of the patches' grid failed");
  }
  const Hit* h = std::min_element(hit, hit + TEAM_MAX, [](const Hit& a, const Hit& b) { return a.i < b.i; });
  if (h->i != INT64_MAX)
    return fail(CELESTE_E_INVALID, "images %lld and %lld overlap in field %d", (long long)h->j, (long long)h->i,
                pt[h->i].field);
  return CELESTE_OK;
}

int check_patch(const celeste_batch* b, const celeste_fields* f, int64_t i) {
  const celeste_image& im = b->images[i];
  const int fi = f->img_field[i];
  if (fi < 0 || fi >= f->n_fields) return fail(CELESTE_E_INVALID, "image %lld: field index out of range", (long long)i);
  const double ox = im.origin[0], oy = im.origin[1];
  if (ox != std::floor(ox) || oy != std::floor(oy))
    return fail(CELESTE_E_INVALID, "image %lld: origin not integer", (long long)i);
  if (ox < 0 || oy < 0 || ox + im.w > f->width || oy + im.h > f->height)
    return fail(CELESTE_E_INVALID, "image %lld: patch outside its field", (long long)i);
  return CELESTE_OK;
}

// patches (may be null) receives where the images lie.
int check_fields(const celeste_batch* b, const Packed& P, const celeste_fields* f, std::vector<Patch>* patches) {
  if (!f || !f->img_field || !f->mean || !f->var) return fail(CELESTE_E_INVALID, "fields and its arrays must not be NULL");
  if (b->mem_kind != CELESTE_MEM_DEVICE) return fail(CELESTE_E_INVALID, "crowded fields need CELESTE_MEM_DEVICE");
  if (f->n_fields < 1 || f->height < 1 || f->width < 1 || f->reserved != 0)
    return fail(CELESTE_E_INVALID, "bad field dimensions");
  if (patches) patches->resize((size_t)P.n_img);
  const int64_t bad = first_failure(P.n_img, 4, [&](int64_t i) {
    if (check_patch(b, f, i) != CELESTE_OK) return false;
    const celeste_image& im = b->images[i];
    if (patches) (*patches)[i] = Patch{f->img_field[i], (int)im.origin[0], (int)im.origin[1], im.w, im.h};
    return true;
  });
  return bad < P.n_img ? check_patch(b, f, bad) : CELESTE_OK;
}

// Checks estimates in device memory there (th2: a second array, or null); they are read back for the message where
// one is out of range.  The flags are 0 between calls.
int check_device_theta(celeste_ctx* ctx, const Packed& P, const double* th1, const double* th2, hipStream_t st) {
  const double* th[2] = {th1, th2};
  if (!ctx->theta_flag.p) {
    CHK(ensure(ctx->theta_flag, sizeof(int) * 2));
    HIPCHK(launch_zero_int(as<int>(ctx->theta_flag), 2, st));
  }
  CHK(ensure_host(ctx->h_flags, sizeof(int) * 2));
  for (int k = 0; k < 2; ++k)
    if (th[k]) HIPCHK(launch_check_theta(th[k], P.n_src, as<int>(ctx->theta_flag) + k, st));
  HIPCHK(hipMemcpyAsync(ctx->h_flags.p, ctx->theta_flag.p, sizeof(int) * 2, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  const int* bad = as<int>(ctx->h_flags);
  if (!bad[0] && !bad[1]) return CELESTE_OK;
  HIPCHK(launch_zero_int(as<int>(ctx->theta_flag), 2, st));
  return theta_error(bad[0] ? th1 : th2, (size_t)P.n_src, st);
}

// The images whose patch meets each RT x RT tile of the fields, in image order: offsets (n_tiles + 1) and, behind
// them, the lists, into ctx->tile_off.  The fields are shared out over host threads.  Lists of up to LIST_PINNED
// bytes are formed in the context's pinned memory; larger ones on the heap, for this call.
constexpr int RT = 32;
constexpr size_t LIST_PINNED = (size_t)8 << 20;
int tile_lists(celeste_ctx* ctx, const std::vector<Patch>& pt, int n_fields, int tx, int tpf, hipStream_t st) {
  const int64_t n = (int64_t)pt.size();
  const int n_tiles = tpf * n_fields;
  std::vector<int> pos((size_t)n_tiles, 0);   // counts, then the next place of each tile
  std::unique_ptr<int[]> heap;
  size_t n_ints = 0;
  int* out = nullptr;
  int rc = CELESTE_OK;
  team(std::min(team_size(n, 80), n_fields), [&](int t, int nt, Barrier& bar) {
    const int f0 = (int)((int64_t)n_fields * t / nt), f1 = (int)((int64_t)n_fields * (t + 1) / nt);
    const auto each = [&](auto fn) {
      for (int64_t i = 0; i < n; ++i) {
        const Patch& p = pt[i];
        if (p.field < f0 || p.field >= f1) continue;
        for (int yy = p.y / RT; yy <= (p.y + p.h - 1) / RT; ++yy)
          for (int xx = p.x / RT; xx <= (p.x + p.w - 1) / RT; ++xx) fn(p.field * tpf + yy * tx + xx, (int)i);
      }
    };
    each([&](int tile, int) { pos[tile] += 1; });
    bar.wait();
    if (t == 0) {
      int64_t total = 0;
      for (int k = 0; k < n_tiles; ++k) total += pos[k];
      n_ints = (size_t)n_tiles + 1 + (size_t)total;
      if (total > INT32_MAX) {
        rc = fail(CELESTE_E_INVALID, "too many patch tiles");
      } else if (n_ints * sizeof(int) <= LIST_PINNED) {
        rc = ensure_host(ctx->h_lists, n_ints * sizeof(int));
        out = as<int>(ctx->h_lists);
      } else {
        heap.reset(new (std::nothrow) int[n_ints]);
        out = heap.get();
        if (!out) rc = fail(CELESTE_E_NOMEM, "host allocation of %zu bytes failed", n_ints * sizeof(int));
      }
      if (rc == CELESTE_OK) {
        int at = 0;
        for (int k = 0; k < n_tiles; ++k) {
          out[k] = at;
          at += pos[k];
          pos[k] = out[k];
        }
        out[n_tiles] = at;
      }
    }
    bar.wait();
    if (rc == CELESTE_OK) each([&](int tile, int i) { out[(size_t)n_tiles + 1 + pos[tile]++] = i; });
  });
  CHK(rc);
  CHK(ensure(ctx->tile_off, n_ints * sizeof(int)));
  if (heap) {
    constexpr size_t W = (size_t)1 << 20;
    const size_t rows = n_ints / W;
    std::vector<Part> parts;
    if (rows) parts.push_back(Part{out, W, 0, (int)rows, (int)W});
    if (n_ints % W) parts.push_back(Part{out + rows * W, W, rows * W, 1, (int)(n_ints % W)});
    return ring_upload(ctx, parts, n_ints, ctx->tile_off.p, st);
  }
  HIPCHK(hipMemcpyAsync(ctx->tile_off.p, out, n_ints * sizeof(int), hipMemcpyHostToDevice, st));
  return CELESTE_OK;
}

}  // namespace

extern "C" {

int celeste_render_fields(celeste_ctx* ctx, const celeste_batch* b, const double* theta, const celeste_fields* f) {
  Packed P;
  std::vector<Patch> patches;
  CHK(validate_and_pack(ctx, b, &P, nullptr, Pack::kNoItems));
  CHK(check_fields(b, P, f, &patches));
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  if (!theta) return fail(CELESTE_E_INVALID, "theta is NULL");
  CHK(check_device_theta(ctx, P, theta, nullptr, st));
  const int tx = (f->width + RT - 1) / RT, ty = (f->height + RT - 1) / RT;
  const int64_t n_tiles64 = (int64_t)tx * ty * f->n_fields;
  if ((int64_t)tx * ty > INT32_MAX || n_tiles64 > INT32_MAX / 2) return fail(CELESTE_E_INVALID, "too many tiles");
  const int n_tiles = (int)n_tiles64, tpf = tx * ty;
  // the metadata and the setup tables are under way while the lists are formed
  CHK(prepare(ctx, b, &P, st, false));
  HIPCHK(launch_setup(as<ImgDev>(ctx->imgs), P.n_img, theta, nullptr, P.prof, as<float>(ctx->tables), P.tstride, st, false));
  const int rc = tile_lists(ctx, patches, f->n_fields, tx, tpf, st);
  if (rc != CELESTE_OK) {
    (void)hipStreamSynchronize(st);   // the pinned metadata is free again
    return rc;
  }
  const int* off = as<int>(ctx->tile_off);
  HIPCHK(launch_render(off, off + n_tiles + 1, n_tiles, as<ImgDev>(ctx->imgs), as<float>(ctx->tables),
                       P.tstride, P.prof.n_exp, P.prof.n_dev, f->height, f->width, tx, tpf, ctx->e_zero, f->mean,
                       f->var, st));
  HIPCHK(hipStreamSynchronize(st));
  return CELESTE_OK;
}

int celeste_neighbour_arrays(celeste_ctx* ctx, const celeste_batch* b, const double* theta, const celeste_fields* f,
                             const int64_t* nbr_off, float* nbr_mean, float* nbr_var) {
  Packed P;
  CHK(validate_and_pack(ctx, b, &P, nullptr, Pack::kNoItems));
  CHK(check_fields(b, P, f, nullptr));
  if (!nbr_off || !nbr_mean || !nbr_var) return fail(CELESTE_E_INVALID, "neighbour arrays must not be NULL");
  for (int i = 0; i < P.n_img; ++i)
    if (nbr_off[i] < 0) return fail(CELESTE_E_INVALID, "negative neighbour offset");
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  if (!theta) return fail(CELESTE_E_INVALID, "theta is NULL");
  CHK(check_device_theta(ctx, P, theta, nullptr, st));
  CHK(ensure(ctx->img_field, sizeof(int) * P.n_img));
  CHK(ensure(ctx->nbr_off, sizeof(long long) * P.n_img));
  CHK(prepare(ctx, b, &P, st, false));
  HIPCHK(hipMemcpyAsync(ctx->img_field.p, f->img_field, sizeof(int) * P.n_img, hipMemcpyHostToDevice, st));
  HIPCHK(hipMemcpyAsync(ctx->nbr_off.p, nbr_off, sizeof(long long) * P.n_img, hipMemcpyHostToDevice, st));
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  HIPCHK(launch_setup(imgs, P.n_img, theta, nullptr, P.prof, as<float>(ctx->tables), P.tstride, st, false));
  HIPCHK(launch_neighbours(imgs, P.n_img, as<int>(ctx->img_field), as<float>(ctx->tables), P.tstride, P.prof.n_exp,
                           P.prof.n_dev, f->height, f->width, ctx->e_zero, f->mean, f->var,
                           as<long long>(ctx->nbr_off), nbr_mean, nbr_var, st));
  HIPCHK(hipStreamSynchronize(st));
  return CELESTE_OK;
}

int celeste_colour_sources(const celeste_batch* b, int32_t* colour, int32_t* n_colours) {
  if (!b || !b->image_offsets || !b->images) return fail(CELESTE_E_INVALID, "batch is NULL or incomplete");
  if (!colour || !n_colours) return fail(CELESTE_E_INVALID, "colour and n_colours must not be NULL");
  if (b->n_sources < 1) return fail(CELESTE_E_INVALID, "n_sources must be >= 1");
  std::vector<Box> box;
  CHK(source_boxes(b, &box));
  const int S = b->n_sources;
  std::unordered_map<int64_t, std::vector<int>> grid;
  std::vector<int> stamp;   // stamp[c] == s: colour c is taken by a neighbour of s
  int nc = 0;
  for (int s = 0; s < S; ++s) {
    const Box& a = box[s];
    for (int64_t cy = a.y0 / CELL; cy <= (a.y1 - 1) / CELL; ++cy)
      for (int64_t cx = a.x0 / CELL; cx <= (a.x1 - 1) / CELL; ++cx) {
        auto it = grid.find(cell_key(cx, cy));
        if (it == grid.end()) continue;
        for (int t : it->second)
          if (overlap(a, box[t])) stamp[colour[t]] = s;
      }
    int c = 0;
    while (c < nc && stamp[c] == s) ++c;
    if (c == nc) {
      ++nc;
      stamp.push_back(-1);
    }
    colour[s] = c;
    for (int64_t cy = a.y0 / CELL; cy <= (a.y1 - 1) / CELL; ++cy)
      for (int64_t cx = a.x0 / CELL; cx <= (a.x1 - 1) / CELL; ++cx) grid[cell_key(cx, cy)].push_back(s);
  }
  *n_colours = nc;
  return CELESTE_OK;
}

int celeste_update_fields(celeste_ctx* ctx, const celeste_batch* b, const double* theta_old, const double* theta_new,
                          const celeste_fields* f) {
  Packed P;
  std::vector<Patch> patches;
  CHK(validate_and_pack(ctx, b, &P, nullptr, Pack::kNoItems));
  CHK(check_fields(b, P, f, &patches));
  CHK(check_disjoint(patches, f->n_fields));
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  if (theta_old && !theta_new) CHK(check_device_theta(ctx, P, theta_old, nullptr, st));   // its error comes first
  if (!theta_old || !theta_new) return fail(CELESTE_E_INVALID, "theta is NULL");
  CHK(check_device_theta(ctx, P, theta_old, theta_new, st));
  CHK(ensure(ctx->tables2, sizeof(float) * (size_t)P.tstride * P.n_img));
  CHK(ensure(ctx->img_field, sizeof(int) * P.n_img));
  CHK(prepare(ctx, b, &P, st, false));
  HIPCHK(hipMemcpyAsync(ctx->img_field.p, f->img_field, sizeof(int) * P.n_img, hipMemcpyHostToDevice, st));
  const ImgDev* imgs = as<ImgDev>(ctx->imgs);
  HIPCHK(launch_setup(imgs, P.n_img, theta_old, nullptr, P.prof, as<float>(ctx->tables), P.tstride, st, false));
  HIPCHK(launch_setup(imgs, P.n_img, theta_new, nullptr, P.prof, as<float>(ctx->tables2), P.tstride, st, false));
  HIPCHK(launch_update_fields(imgs, P.n_img, as<int>(ctx->img_field), as<float>(ctx->tables),
                              as<float>(ctx->tables2), P.tstride, P.prof.n_exp, P.prof.n_dev, f->height, f->width,
                              ctx->e_zero, f->mean, f->var, st));
  HIPCHK(hipStreamSynchronize(st));
  return CELESTE_OK;
}

int celeste_field_elbo(celeste_ctx* ctx, const celeste_batch* b, const double* theta, const celeste_fields* f,
                       const float* field_pixels, const double* field_sky, double* elbo_out) {
  Packed P;
  CHK(validate_and_pack(ctx, b, &P, nullptr, Pack::kCheck));
  CHK(check_fields(b, P, f, nullptr));
  if (!field_pixels || !field_sky || !elbo_out)
    return fail(CELESTE_E_INVALID, "field_pixels, field_sky and elbo_out must not be NULL");
  for (int k = 0; k < f->n_fields; ++k)
    if (!(field_sky[k] > 0.0) || !std::isfinite(field_sky[k]))
      return fail(CELESTE_E_INVALID, "field %d: sky must be finite and > 0", k);
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  if (!theta) return fail(CELESTE_E_INVALID, "theta is NULL");
  CHK(check_device_theta(ctx, P, theta, nullptr, st));
  const int S = P.n_src;
  const int64_t n = (int64_t)f->n_fields * f->height * f->width;
  const int per_block = 8192;
  const int64_t nb64 = (n + per_block - 1) / per_block;
  if (nb64 > INT32_MAX / 2) return fail(CELESTE_E_INVALID, "fields too large");
  const int nb = (int)nb64;
  CHK(ensure(ctx->fsky, sizeof(double) * f->n_fields));
  CHK(ensure(ctx->o_elbo, sizeof(double) * S));
  CHK(ensure(ctx->partials, sizeof(double) * (size_t)nb));
  HIPCHK(hipMemcpyAsync(ctx->fsky.p, field_sky, sizeof(double) * f->n_fields, hipMemcpyHostToDevice, st));
  HIPCHK(launch_prior_term(theta, S, P.prior, as<double>(ctx->o_elbo), st));
  HIPCHK(launch_field_terms(field_pixels, f->mean, f->var, as<double>(ctx->fsky), f->height, f->width, f->n_fields,
                            per_block, nb, as<double>(ctx->partials), st));
  std::vector<double> pri(S), part(nb);
  HIPCHK(hipMemcpyAsync(pri.data(), ctx->o_elbo.p, sizeof(double) * S, hipMemcpyDeviceToHost, st));
  HIPCHK(hipMemcpyAsync(part.data(), ctx->partials.p, sizeof(double) * nb, hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  double tot = 0.0;
  for (double v : part) tot += v;
  for (double v : pri) tot += v;
  *elbo_out = tot;
  return CELESTE_OK;
}

int celeste_start(celeste_ctx* ctx, const celeste_batch* b, double* theta_inout, const celeste_fit_opts* opts,
                  double* elbo_out) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  return run_fit(ctx, b, theta_inout, opts, nullptr, ctx->stream, true, elbo_out, true);
}

}  // extern "C"

// =============================================================================== autotuner

namespace {

std::string tune_key(celeste_ctx* ctx, const Packed& P, const celeste_batch* b) {
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, ctx->device) != hipSuccess) std::memset(&prop, 0, sizeof(prop));
  int max_psf = 1;
  double px = 0.0;
  for (int i = 0; i < P.n_img; ++i) {
    max_psf = std::max(max_psf, b->images[i].n_psf);
    px += (double)b->images[i].h * b->images[i].w;
  }
  const int cls = (int)std::lround(std::log2(std::max(1.0, px / std::max(1, P.n_img))));
  char buf[512];
  std::snprintf(buf, sizeof(buf), "%s|%s|cu%d|exp%d|dev%d|psf%d|px2^%d", prop.name, prop.gcnArchName,
                prop.multiProcessorCount, P.prof.n_exp, P.prof.n_dev, max_psf, cls);
  std::string k(buf);
  for (char& c : k)
    if (c == ' ' || c == '\t' || c == '\n') c = '_';
  return k;
}

// 1 if the cache holds the key (fills r), 0 if not or the file does not exist yet.
int tune_cache_read(const char* path, const std::string& key, celeste_tune_result* r) {
  FILE* f = std::fopen(path, "r");
  if (!f) return 0;
  char line[1024];
  int found = 0;
  while (std::fgets(line, sizeof(line), f)) {
    char k[600];
    celeste_tune_result t{};
    if (std::sscanf(line, "%599s %d %d %d %d %d %d %lf %lf", k, &t.chunk_px, &t.block, &t.variant, &t.tile_w,
                    &t.value_block, &t.value_tile_w, &t.full_ms, &t.value_ms) == 9 &&
        key == k) {
      *r = t;   // the last matching line wins
      found = 1;
    }
  }
  std::fclose(f);
  return found;
}

int tune_cache_append(const char* path, const std::string& key, const celeste_tune_result& r) {
  FILE* f = std::fopen(path, "a");
  if (!f) return fail(CELESTE_E_INVALID, "autotune cache %s: cannot open for appending", path);
  std::fprintf(f, "%s %d %d %d %d %d %d %.6f %.6f\n", key.c_str(), r.chunk_px, r.block, r.variant, r.tile_w,
               r.value_block, r.value_tile_w, r.full_ms, r.value_ms);
  std::fclose(f);
  return CELESTE_OK;
}

int log2_tile(int w) {
  for (int k = 3; k <= 6; ++k)
    if (w == (1 << k)) return k;
  return -1;
}

// Minimum over `reps` timed launches (after one untimed) of a launch sequence, in ms.
template <class F>
int time_min(hipStream_t st, int reps, F launch, double* best) {
  hipEvent_t a = nullptr, z = nullptr;
  HIPCHK(hipEventCreate(&a));
  HIPCHK(hipEventCreate(&z));
  int rc = CELESTE_OK;
  *best = 1e300;
  for (int r = 0; r <= reps && rc == CELESTE_OK; ++r) {
    hipError_t e = hipEventRecord(a, st);
    if (e == hipSuccess) e = launch();
    if (e == hipSuccess) e = hipEventRecord(z, st);
    if (e == hipSuccess) e = hipEventSynchronize(z);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, z);
    if (e != hipSuccess) rc = fail(CELESTE_E_DEVICE, "autotune launch: %s", hipGetErrorString(e));
    else if (r > 0) *best = std::min(*best, (double)ms);
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(z);
  return rc;
}

int autotune(celeste_ctx* ctx, const celeste_batch* b, const double* theta, int64_t sample_px,
             const char* cache_path, celeste_tune_result* out) {
  if (!ctx) return fail(CELESTE_E_INVALID, "context is NULL");
  if (!theta) return fail(CELESTE_E_INVALID, "theta is NULL");
  Packed P0;
  CHK(validate_and_pack(ctx, b, &P0));
  HIPCHK(hipSetDevice(ctx->device));
  const hipStream_t st = ctx->stream;
  const std::string key = tune_key(ctx, P0, b);
  celeste_tune_result r{};
  if (cache_path && tune_cache_read(cache_path, key, &r)) {
    const int tl = log2_tile(r.tile_w), vl = log2_tile(r.value_tile_w);
    if (tl < 0 || vl < 0 || (r.block != 128 && r.block != 256) || (r.value_block != 128 && r.value_block != 256) ||
        r.variant < 0 || r.variant > 7 || r.chunk_px < 64 || r.chunk_px > (1 << 24))
      return fail(CELESTE_E_INVALID, "autotune cache %s: bad entry for %s", cache_path, key.c_str());
    ctx->chunk_px = r.chunk_px;
    ctx->block = r.block;
    ctx->variant = r.variant;
    ctx->tile_log2 = tl;
    ctx->vblock = r.value_block;
    ctx->vtile_log2 = vl;
    r.from_cache = 1;
    if (out) *out = r;
    return CELESTE_OK;
  }
  // theta on the host, for the sample
  const int S = b->n_sources;
  std::vector<double> th((size_t)S * NP);
  if (b->mem_kind == CELESTE_MEM_HOST)
    std::memcpy(th.data(), theta, sizeof(double) * th.size());
  else {
    HIPCHK(hipMemcpyAsync(th.data(), theta, sizeof(double) * th.size(), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
  }
  for (int s = 0; s < S; ++s) CHK(check_theta(th.data() + (size_t)s * NP, s));
  // every k-th source, about sample_px pixels
  if (sample_px <= 0) sample_px = 60000000;
  int64_t total = 0;
  for (int64_t i = 0; i < b->image_offsets[S]; ++i) total += (int64_t)b->images[i].h * b->images[i].w;
  const int64_t stride = std::max<int64_t>(1, total / std::max<int64_t>(1, sample_px));
  std::vector<int64_t> offs{0};
  std::vector<celeste_image> imgs;
  std::vector<double> ths;
  for (int64_t s = 0; s < S; s += stride) {
    for (int64_t i = b->image_offsets[s]; i < b->image_offsets[s + 1]; ++i) {
      imgs.push_back(b->images[i]);
      r.sample_px += (int64_t)b->images[i].h * b->images[i].w;
    }
    offs.push_back((int64_t)imgs.size());
    ths.insert(ths.end(), th.begin() + s * NP, th.begin() + (s + 1) * NP);
  }
  r.sample_sources = (int64_t)offs.size() - 1;
  celeste_batch sub = *b;
  sub.n_sources = (int32_t)r.sample_sources;
  sub.image_offsets = offs.data();
  sub.images = imgs.data();
  CHK(ensure(ctx->theta, sizeof(double) * ths.size()));
  HIPCHK(hipMemcpyAsync(ctx->theta.p, ths.data(), sizeof(double) * ths.size(), hipMemcpyHostToDevice, st));
  const double* th_dev = as<double>(ctx->theta);

  // every return before the end leaves the context's work-item size as it was
  struct ChunkGuard {
    celeste_ctx* c;
    int saved;
    ~ChunkGuard() { c->chunk_px = saved; }
  } guard{ctx, ctx->chunk_px};
  const int chunks[] = {4096, 8192, 16384};
  const int variants[] = {2, 3, 6, 7};
  struct Cand {
    double ms;
    int chunk, block, variant, tl;
    bool is_default() const { return chunk == 4096 && block == 256 && variant == 3 && tl == 3; }
  };
  std::vector<Cand> cands;
  int rc = CELESTE_OK;
  for (int chunk : chunks) {
    ctx->chunk_px = chunk;
    Packed P;
    rc = validate_and_pack(ctx, &sub, &P);
    if (rc == CELESTE_OK) rc = prepare(ctx, &sub, &P, st);
    if (rc != CELESTE_OK) break;
    const ImgDev* di = as<ImgDev>(ctx->imgs);
    float* tables = as<float>(ctx->tables);
    HIPCHK(launch_setup(di, P.n_img, th_dev, nullptr, P.prof, tables, P.tstride, st));
    for (int block : {128, 256})
      for (int variant : variants)
        for (int tl = 3; tl <= 6 && rc == CELESTE_OK; ++tl) {
          double ms = 0.0;
          rc = time_min(st, 3, [&]() {
            return launch_eval_full(as<WorkItem>(ctx->items), P.n_items, di, tables, P.tstride, P.prof.n_exp,
                                    P.prof.n_dev, nullptr, as<double>(ctx->partials), block,
                                    variant | (ctx->fp64_sums ? 8 : 0), tl, ctx->e_zero, st);
          }, &ms);
          r.n_candidates += 1;
          double& unit_best = (variant & 4) ? r.matrix_full_ms : r.vector_full_ms;
          if (rc == CELESTE_OK && (unit_best == 0.0 || ms < unit_best)) unit_best = ms;
          if (rc == CELESTE_OK) cands.push_back(Cand{ms, chunk, block, variant, tl});
        }
    if (rc != CELESTE_OK) break;
  }
  if (rc != CELESTE_OK) return rc;
  if (cands.empty()) return fail(CELESTE_E_DEVICE, "autotune: no candidate could be timed");
  // the four fastest and the default again, nine launches each, in one pass: candidates within a
  // few per cent of each other are ordered by more than one noisy minimum, and the default is
  // timed beside them, so the pick is never slower than the default by the pass's own timings
  std::sort(cands.begin(), cands.end(), [](const Cand& x, const Cand& y) { return x.ms < y.ms; });
  {
    std::vector<Cand> fin(cands.begin(), cands.begin() + std::min<size_t>(4, cands.size()));
    bool has_default = false;
    for (const Cand& c : fin) has_default = has_default || c.is_default();
    if (!has_default)
      for (const Cand& c : cands)
        if (c.is_default()) fin.push_back(c);
    cands.swap(fin);
  }
  std::stable_sort(cands.begin(), cands.end(), [](const Cand& x, const Cand& y) { return x.chunk < y.chunk; });
  {
    int prepared = 0;
    Packed P;
    for (Cand& c : cands) {
      if (c.chunk != prepared) {
        ctx->chunk_px = c.chunk;
        CHK(validate_and_pack(ctx, &sub, &P));
        CHK(prepare(ctx, &sub, &P, st));
        HIPCHK(launch_setup(as<ImgDev>(ctx->imgs), P.n_img, th_dev, nullptr, P.prof, as<float>(ctx->tables),
                            P.tstride, st));
        prepared = c.chunk;
      }
      const ImgDev* di = as<ImgDev>(ctx->imgs);
      float* tables = as<float>(ctx->tables);
      CHK(time_min(st, 9, [&]() {
        return launch_eval_full(as<WorkItem>(ctx->items), P.n_items, di, tables, P.tstride, P.prof.n_exp,
                                P.prof.n_dev, nullptr, as<double>(ctx->partials), c.block,
                                c.variant | (ctx->fp64_sums ? 8 : 0), c.tl, ctx->e_zero, st);
      }, &c.ms));
      if (c.is_default()) r.default_full_ms = c.ms;
    }
  }
  {
    // fastest of the pass; on a tie the default stays
    const Cand* pick = nullptr;
    for (const Cand& c : cands)
      if (!pick || c.ms < pick->ms || (c.ms == pick->ms && c.is_default())) pick = &c;
    r.full_ms = pick->ms;
    r.chunk_px = pick->chunk;
    r.block = pick->block;
    r.variant = pick->variant;
    r.tile_w = 1 << pick->tl;
  }
  // value kernel on the chosen work items
  ctx->chunk_px = r.chunk_px;
  {
    Packed P;
    CHK(validate_and_pack(ctx, &sub, &P));
    CHK(prepare(ctx, &sub, &P, st));
    const ImgDev* di = as<ImgDev>(ctx->imgs);
    float* tables = as<float>(ctx->tables);
    HIPCHK(launch_setup(di, P.n_img, th_dev, nullptr, P.prof, tables, P.tstride, st));
    double vbest = 1e300;
    for (int vblock : {128, 256})
      for (int tl = 3; tl <= 6; ++tl) {
        double ms = 0.0;
        CHK(time_min(st, 3, [&]() {
          return launch_eval_value(as<WorkItem>(ctx->items), P.n_items, di, tables, P.tstride, P.prof.n_exp,
                                   P.prof.n_dev, nullptr, as<double>(ctx->partials), vblock, r.variant, tl,
                                   ctx->e_zero, st);
        }, &ms));
        r.n_candidates += 1;
        if (vblock == 256 && tl == 3 && r.chunk_px == 4096) r.default_value_ms = ms;
        if (ms < vbest) {
          vbest = ms;
          r.value_ms = ms;
          r.value_block = vblock;
          r.value_tile_w = 1 << tl;
        }
      }
  }
  if (r.chunk_px != 4096) {
    // the default's value-kernel time on its own work items
    ctx->chunk_px = 4096;
    Packed P;
    CHK(validate_and_pack(ctx, &sub, &P));
    CHK(prepare(ctx, &sub, &P, st));
    const ImgDev* di = as<ImgDev>(ctx->imgs);
    float* tables = as<float>(ctx->tables);
    HIPCHK(launch_setup(di, P.n_img, th_dev, nullptr, P.prof, tables, P.tstride, st));
    CHK(time_min(st, 3, [&]() {
      return launch_eval_value(as<WorkItem>(ctx->items), P.n_items, di, tables, P.tstride, P.prof.n_exp,
                               P.prof.n_dev, nullptr, as<double>(ctx->partials), 256, 3, 3, ctx->e_zero, st);
    }, &r.default_value_ms));
  }
  guard.saved = r.chunk_px;  // the guard leaves the chosen size on the context
  ctx->block = r.block;
  ctx->variant = r.variant;
  ctx->tile_log2 = log2_tile(r.tile_w);
  ctx->vblock = r.value_block;
  ctx->vtile_log2 = log2_tile(r.value_tile_w);
  if (cache_path) CHK(tune_cache_append(cache_path, key, r));
  if (out) *out = r;
  return CELESTE_OK;
}

}  // namespace

extern "C" int celeste_autotune(celeste_ctx* ctx, const celeste_batch* batch, const double* theta, int64_t sample_px,
                                const char* cache_path, celeste_tune_result* out) {
  return autotune(ctx, batch, theta, sample_px, cache_path, out);
}
