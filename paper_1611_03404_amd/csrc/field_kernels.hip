// Crowded fields: rendering every source's expected counts and their variance into shared
// field images, and the per-source neighbour arrays (section III-B: each source is
// optimised with the other sources held fixed at their current estimates; pixels receive
// photons from several sources).
//
// Rendering is a gather, deterministic by construction: the wavefronts of a 32x32 tile of a
// field walk the list of source patches overlapping the tile in source order and sum
// their contributions in FP64 per pixel.  The neighbour array of a source is the rendered
// field minus the source's own contribution, computed by the same per-pixel routine (Mixture::rates, whose
// operations are written out so that every kernel rounds them alike).
#include <algorithm>

#include "celeste_internal.h"
#include "tiles.h"

namespace celeste {

namespace {

using namespace tab;

constexpr int RTILE = 32;   // side of the tiles that the host lists sources for

// Which components of a source can be non-zero on a 64-pixel tile: a bit per galaxy component, and one
// per PSF component for the star.
struct TileHits {
  unsigned long long gal;
  unsigned star;
};

// A source's mixture on one image, as a wavefront's tiles need it: the skip test of one component per
// lane (the star's components after the galaxy's; where they do not all fit, the star's are not tested).
template <int NE, int ND>
struct Mixture {
  const float* __restrict__ T;
  int npsf, n_exp, ncomp, n_gal;
  float psx, psy;
  SkipTest skip;

  __device__ __forceinline__ Mixture(const float* __restrict__ T_, int npsf_, int n_exp_, int n_dev_, int lane)
      : T(T_), npsf(npsf_), n_exp(NE > 0 ? NE : n_exp_), ncomp(NE > 0 ? NE + ND : n_exp_ + n_dev_) {
    n_gal = npsf * ncomp;   // at most 64
    psx = T[PSX];
    psy = T[PSY];
    const int c = min(lane, n_gal - 1), k = lane - n_gal;
    const bool star = k >= 0;
    const float* sr = T + STAR + STAR_REC * (star ? min(k, npsf - 1) : c / ncomp);
    skip = skip_test(star ? sr : T + EXPO + c * EXPO_REC, sr, 0.f);
  }

  __device__ __forceinline__ TileHits split(unsigned long long hits) const {
    TileHits h;
    h.gal = hits & lane_mask(n_gal);
    const unsigned all = (1u << npsf) - 1;
    h.star = n_gal + npsf <= 64 ? (unsigned)(hits >> (n_gal & 63)) & all : all;
    return h;
  }

  // Expected counts e = calib T and variance v = calib^2 U of the source at one pixel per lane for each of Q
  // tiles, (dx0, dy0) from the source in patch coordinates.  Every tile sees the operations of a sum
  // over all components in order: a component that is left out adds exactly 0.
  template <int Q>
  __device__ __forceinline__ void rates(const TileHits (&h)[Q], const float (&dx0)[Q], const float (&dy0)[Q],
                                        float (&e)[Q], float (&v)[Q]) const {
#pragma clang fp contract(off)
    float Gs[Q], gx[Q], gd[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) Gs[q] = gx[q] = gd[q] = 0.f;
    for (int k = 0; k < npsf; ++k) {
      unsigned hk[Q], any = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        hk[q] = (unsigned)(h[q].gal >> (k * ncomp)) & (unsigned)lane_mask(min(32, ncomp));
        any |= hk[q] | ((h[q].star >> k) & 1u);
      }
      if (!any) continue;
      const float* __restrict__ sr = T + STAR + k * STAR_REC;
      const float* __restrict__ Ek = T + EXPO + k * ncomp * EXPO_REC;
      const float xix = sr[S_XIX], xiy = sr[S_XIY];
      const ValRec st = load_val(sr);
      if constexpr (NE > 0) {
        ExpoBlock<NE> vx;
        ExpoBlock<ND> vd;
        vx.load(Ek);
        vd.load(Ek + NE * EXPO_REC);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const float dx = dx0[q] - xix, dy = dy0[q] - xiy;
          const float dxx = dx * dx, dxy = dx * dy, dyy = dy * dy;
          if ((h[q].star >> k) & 1u) comp_value(st, dxx, dxy, dyy, Gs[q]);
          if (!hk[q]) continue;
#pragma unroll
          for (int j = 0; j < NE; j += 2)
            if (hk[q] & (3u << j)) {
              comp_value(vx.rec(j), dxx, dxy, dyy, gx[q]);
              if (j + 1 < NE) comp_value(vx.rec(j + 1), dxx, dxy, dyy, gx[q]);
            }
#pragma unroll
          for (int j = 0; j < ND; j += 2)
            if ((hk[q] >> NE) & (3u << j)) {
              comp_value(vd.rec(j), dxx, dxy, dyy, gd[q]);
              if (j + 1 < ND) comp_value(vd.rec(j + 1), dxx, dxy, dyy, gd[q]);
            }
        }
      } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const float dx = dx0[q] - xix, dy = dy0[q] - xiy;
          const float dxx = dx * dx, dxy = dx * dy, dyy = dy * dy;
          if ((h[q].star >> k) & 1u) comp_value(st, dxx, dxy, dyy, Gs[q]);
          for (int j = 0; j < ncomp; ++j)
            if ((hk[q] >> j) & 1u) comp_value(load_val(Ek + j * EXPO_REC), dxx, dxy, dyy, j < n_exp ? gx[q] : gd[q]);
        }
      }
    }
    const float ed = T[EDEV], io = T[CALIB], cs = T[CS], cg = T[CG], Ks = T[KS], Kg = T[KG], Ksg = T[KSG];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float Gg = fmaf(ed, gd[q] - gx[q], gx[q]);
      const float Tv = fmaf(cs, Gs[q], cg * Gg);
      const float Uv = fmaf(Ks, Gs[q] * Gs[q], fmaf(Kg, Gg * Gg, Ksg * Gs[q] * Gg));
      e[q] = io * Tv;
      v[q] = io * io * Uv;
    }
  }

  // ... on one tile of a walk over the image
  template <class MAP>
  __device__ __forceinline__ void rate(const MAP& tm, int row, int col, int first, float e_zero, float& e,
                                       float& v) const {
    const TileHits h[1] = {split(tile_hits(skip, tm, col, first, psx, psy, e_zero))};
    const float dx0[1] = {(float)col - psx}, dy0[1] = {(float)row - psy};
    float e1[1], v1[1];
    rates<1>(h, dx0, dy0, e1, v1);
    e = e1[0];
    v = v1[0];
  }
};

// Field images from the sources' patches.  A wavefront takes Q 8 x 8 squares of a tile, the tile's list is read 64
// sources at a time, one per lane, and the wavefront walks those whose patch meets its squares, evaluating
// per square the components that can be non-zero on it (tiles.h; the field's stars and most galaxies are
// exactly 0 over most of a large patch).  Bound by vector issue and by the latency of a source's table:
// its loads serve all Q squares, and the blocks of neighbouring tiles run on one XCD, whose cache
// then holds the tables they share.  60,000 patches (2e8 px) into ten 512 x 512 fields: 2.0 ms
// with Q = 2, 2.15 with 1, 2.1 with 4 (fewer, longer wavefronts); 15.0 ms with every component evaluated on a
// lane per pixel row, a scalar load and a call per pixel each.
constexpr int RQ = 2;

template <int NE, int ND, int Q>
__global__ __launch_bounds__(256) void k_render(const int* __restrict__ tile_off, const int* __restrict__ tile_img,
                                                const ImgDev* __restrict__ imgs, const float* __restrict__ tables,
                                                int tstride, int n_exp, int n_dev, int H, int W, int tiles_x,
                                                int tiles_per_field, int tile0, int n_blocks, float e_zero,
                                                float* __restrict__ mean, float* __restrict__ var) {
  constexpr int QX = Q >= 2 ? 2 : 1, QY = Q / QX;       // squares of a wavefront
  constexpr int BX = RTILE / (16 * QX), BY = RTILE / (16 * QY);   // blocks of a tile
  const int per_xcd = (int)gridDim.x >> 3;
  const int blk = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);   // neighbouring tiles on one XCD
  if (blk >= n_blocks) return;
  const int local = blk / (BX * BY), part = blk - local * (BX * BY), tile = tile0 + local;
  const int f = tile / tiles_per_field, tt = tile - f * tiles_per_field;
  const int ty = tt / tiles_x, tx = tt - ty * tiles_x;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the wavefront's pixels: [px0, px0 + 8 QX) x [py0, py0 + 8 QY)
  const int px0 = tx * RTILE + (part % BX) * (16 * QX) + (wv & 1) * (8 * QX);
  const int py0 = ty * RTILE + (part / BX) * (16 * QY) + (wv >> 1) * (8 * QY);
  const int lx = lane & 7, ly = lane >> 3;
  double e[Q], v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) e[q] = v[q] = 0.0;
  const int q0 = tile_off[tile], q1 = tile_off[tile + 1];
  for (int base = q0; base < q1; base += 64) {
    const bool in = base + lane < q1;
    const int my_img = tile_img[in ? base + lane : q0];
    const ImgDev& im = imgs[my_img];
    const int my_w = im.w, my_h = im.h, my_npsf = im.n_psf;
    const int my_x = px0 - (int)im.origin[0], my_y = py0 - (int)im.origin[1];   // of px0, py0 in the patch
    const bool meets = in && my_x + 8 * QX > 0 && my_x < my_w && my_y + 8 * QY > 0 && my_y < my_h;
    for (unsigned long long todo = __ballot(meets); todo; todo &= todo - 1) {
      const int l = __builtin_ctzll(todo);
      const int i = __builtin_amdgcn_readlane(my_img, l), npsf = __builtin_amdgcn_readlane(my_npsf, l);
      const int w = __builtin_amdgcn_readlane(my_w, l), h = __builtin_amdgcn_readlane(my_h, l);
      const int x = __builtin_amdgcn_readlane(my_x, l), y = __builtin_amdgcn_readlane(my_y, l);
      const Mixture<NE, ND> mix(tables + (size_t)i * tstride, npsf, n_exp, n_dev, lane);
      TileHits hits[Q];
      float dx0[Q], dy0[Q], de[Q], dv[Q];
      bool any = false;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int xq = x + 8 * (q % QX), yq = y + 8 * (q / QX);
        const TileBox b{max(xq, 0), min(xq + 7, w - 1), max(yq, 0), min(yq + 7, h - 1)};
        hits[q] = TileHits{0ull, 0u};
        if (b.x0 <= b.x1 && b.y0 <= b.y1) hits[q] = mix.split(__ballot(may_hit(mix.skip, b, mix.psx, mix.psy, e_zero)));
        any = any || hits[q].gal || hits[q].star;
        dx0[q] = (float)(xq + lx) - mix.psx;
        dy0[q] = (float)(yq + ly) - mix.psy;
      }
      if (!any) continue;
      mix.template rates<Q>(hits, dx0, dy0, de, dv);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int c = x + 8 * (q % QX) + lx, r = y + 8 * (q / QX) + ly;
        const bool inside = (unsigned)c < (unsigned)w && (unsigned)r < (unsigned)h;
        e[q] += (double)(inside ? de[q] : 0.f);
        v[q] += (double)(inside ? dv[q] : 0.f);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int px = px0 + 8 * (q % QX) + lx, py = py0 + 8 * (q / QX) + ly;
    if (px < W && py < H) {
      const size_t o = ((size_t)f * H + py) * W + px;
      mean[o] = (float)e[q];
      var[o] = (float)v[q];
    }
  }
}

// Blocks of 4 wavefronts per patch in k_neighbours and k_update: a batch of few patches ends sooner with two
// than with one, and 4,000 patches of 15..121 px take no longer (1: 122 and 226 us, 2: 126 and 228, 4: 141 and 249).
constexpr int SPLIT = 2;

// Neighbour arrays of one patch image: field totals minus the source's own contribution,
// clamped at zero against rounding.  The tile walk and skips of the pixel kernels: 126 us for 4,000
// patches (1e7 px), 505 us with every component evaluated in rows.
template <int NE, int ND>
__global__ __launch_bounds__(256) void k_neighbours(const ImgDev* __restrict__ imgs, const int* __restrict__ img_field,
                                                    const float* __restrict__ tables, int tstride, int n_exp,
                                                    int n_dev, int H, int W, float e_zero,
                                                    const float* __restrict__ mean, const float* __restrict__ var,
                                                    const long long* __restrict__ nbr_off,
                                                    float* __restrict__ nbr_mean, float* __restrict__ nbr_var) {
  const int i = blockIdx.x, lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + 4 * blockIdx.y;
  const ImgDev& im = imgs[i];
  const int c0 = (int)im.origin[0], r0 = (int)im.origin[1], w = im.w;
  const size_t corner = ((size_t)img_field[i] * H + r0) * W + c0;
  float* om = nbr_mean + nbr_off[i];
  float* ov = nbr_var + nbr_off[i];
  const Mixture<NE, ND> mix(tables + (size_t)i * tstride, im.n_psf, n_exp, n_dev, lane);
  TileMap<true, 4 * SPLIT> tm(WorkItem{i, 0, 0, im.h}, w, im.h, 3, nullptr, wv);
  for (; tm.more(); tm.next()) {
    int row, col, first;
    bool live;
    tm.pixel(lane, row, col, live, first);
    const size_t o = corner + (size_t)row * W + col;
    const float fm = mean[o], fv = var[o];
    float de, dv;
    mix.rate(tm, row, col, first, e_zero, de, dv);
    if (live) {
#pragma clang fp contract(off)
      om[(size_t)row * w + col] = fmaxf(fm - de, 0.f);
      ov[(size_t)row * w + col] = fmaxf(fv - dv, 0.f);
    }
  }
}

// Moves the field images from one estimate of the batch's sources to another: each pixel of
// each patch gets (new - old) contribution of its source.  Patches of one launch must not
// overlap within a field, so every pixel has a single writer.  228 us for 4,000 patches (1e7 px), 1,000 us with
// every component evaluated in rows.
template <int NE, int ND>
__global__ __launch_bounds__(256) void k_update(const ImgDev* __restrict__ imgs, const int* __restrict__ img_field,
                                                const float* __restrict__ t_old, const float* __restrict__ t_new,
                                                int tstride, int n_exp, int n_dev, int H, int W, float e_zero,
                                                float* __restrict__ mean, float* __restrict__ var) {
  const int i = blockIdx.x, lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + 4 * blockIdx.y;
  const ImgDev& im = imgs[i];
  const int c0 = (int)im.origin[0], r0 = (int)im.origin[1];
  const size_t corner = ((size_t)img_field[i] * H + r0) * W + c0;
  const Mixture<NE, ND> was(t_old + (size_t)i * tstride, im.n_psf, n_exp, n_dev, lane);
  const Mixture<NE, ND> is(t_new + (size_t)i * tstride, im.n_psf, n_exp, n_dev, lane);
  TileMap<true, 4 * SPLIT> tm(WorkItem{i, 0, 0, im.h}, im.w, im.h, 3, nullptr, wv);
  for (; tm.more(); tm.next()) {
    int row, col, first;
    bool live;
    tm.pixel(lane, row, col, live, first);
    const size_t o = corner + (size_t)row * W + col;
    const float fm = mean[o], fv = var[o];
    float eo, vo, en, vn;
    was.rate(tm, row, col, first, e_zero, eo, vo);
    is.rate(tm, row, col, first, e_zero, en, vn);
    if (live) {
#pragma clang fp contract(off)
      mean[o] = fmaxf(fm + (en - eo), 0.f);
      var[o] = fmaxf(fv + (vn - vo), 0.f);
    }
  }
}

// Delta-method expected log-likelihood of every field pixel in FP64 (E = sky + mean,
// Var = var), one partial sum per block.
__global__ __launch_bounds__(256) void k_field_terms(const float* __restrict__ x, const float* __restrict__ mean,
                                                     const float* __restrict__ var,
                                                     const double* __restrict__ sky, int H, int W, int n_fields,
                                                     int per_block, double* __restrict__ partials) {
  __shared__ double red[4];
  const size_t npf = (size_t)H * W, n = npf * n_fields;
  const size_t b0 = (size_t)blockIdx.x * per_block;
  double acc = 0.0;
  for (size_t k = b0 + threadIdx.x; k < b0 + per_block && k < n; k += 256) {
    const double xv = x[k], E = sky[k / npf] + (double)mean[k], V = var[k];
    acc += xv * (log(E) - V / (2.0 * E * E)) - E - lgamma(xv + 1.0);
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// The instances with the standard profiles' component counts unrolled (as in the pixel kernels).
bool unrolled(int n_exp, int n_dev) { return n_exp == 6 && n_dev == 8; }

}  // namespace

hipError_t launch_update_fields(const ImgDev* imgs, int n_img, const int* img_field, const float* t_old,
                                const float* t_new, int tstride, int n_exp, int n_dev, int H, int W,
                                float e_zero, float* mean, float* var, hipStream_t st) {
  if (n_img <= 0) return hipSuccess;
  const auto k = unrolled(n_exp, n_dev) ? &k_update<6, 8> : &k_update<0, 0>;
  hipLaunchKernelGGL(k, dim3(n_img, SPLIT), dim3(256), 0, st, imgs, img_field, t_old, t_new, tstride, n_exp, n_dev, H,
                     W, e_zero, mean, var);
  return hipGetLastError();
}

hipError_t launch_field_terms(const float* x, const float* mean, const float* var, const double* sky, int H, int W,
                              int n_fields, int per_block, int n_blocks, double* partials, hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_field_terms, dim3(n_blocks), dim3(256), 0, st, x, mean, var, sky, H, W, n_fields, per_block,
                     partials);
  return hipGetLastError();
}

hipError_t launch_render(const int* tile_off, const int* tile_img, int n_tiles, const ImgDev* imgs,
                         const float* tables, int tstride, int n_exp, int n_dev, int H, int W, int tiles_x,
                         int tiles_per_field, float e_zero, float* mean, float* var, hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  const auto k = unrolled(n_exp, n_dev) ? &k_render<6, 8, RQ> : &k_render<0, 0, RQ>;
  // A launch holds fewer than 2^32 threads; one with more runs some of its blocks only, without an error.
  constexpr int PER_LAUNCH = 1 << 22;
  for (int t0 = 0; t0 < n_tiles; t0 += std::min(PER_LAUNCH, n_tiles - t0)) {
    const int n_blocks = std::min(PER_LAUNCH, n_tiles - t0) * (4 / RQ);
    hipLaunchKernelGGL(k, dim3((n_blocks + 7) / 8 * 8), dim3(256), 0, st, tile_off, tile_img, imgs, tables, tstride,
                       n_exp, n_dev, H, W, tiles_x, tiles_per_field, t0, n_blocks, e_zero, mean, var);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_neighbours(const ImgDev* imgs, int n_img, const int* img_field, const float* tables, int tstride,
                             int n_exp, int n_dev, int H, int W, float e_zero, const float* mean, const float* var,
                             const long long* nbr_off, float* nbr_mean, float* nbr_var, hipStream_t st) {
  if (n_img <= 0) return hipSuccess;
  const auto k = unrolled(n_exp, n_dev) ? &k_neighbours<6, 8> : &k_neighbours<0, 0>;
  hipLaunchKernelGGL(k, dim3(n_img, SPLIT), dim3(256), 0, st, imgs, img_field, tables, tstride, n_exp, n_dev, H, W,
                     e_zero, mean, var, nbr_off, nbr_mean, nbr_var);
  return hipGetLastError();
}

}  // namespace celeste
