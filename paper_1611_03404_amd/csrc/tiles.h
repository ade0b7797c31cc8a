// Pixel tiles of the mixture kernels: the pixel -> lane layout of a work item, and the test that
// decides for a whole tile which mixture components can be non-zero on it.
#pragma once

#include "celeste_internal.h"

namespace celeste {
namespace {

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// Pixel box of a tile: columns [x0, x1], rows [y0, y1] (wave-uniform).
struct TileBox {
  int x0, x1, y0, y1;
};

// A pointer read from a metadata record, known to be device memory: its loads are global loads.  (Through
// a plain pointer they are flat loads, which count as scalar-memory operations too, so that every wait
// for a table record also waits for the pixels.)
typedef const __attribute__((address_space(1))) float* GlobalF;
__device__ __forceinline__ GlobalF global(const float* p) { return (GlobalF)p; }

// The pixels of an image and, where given, its neighbour arrays.  (A second address form for images whose
// byte offsets fit in 32 bits, one 24-bit multiply-add instead of a 64-bit product, was slower: the
// scalars it holds cost the value+gradient+Hessian kernel more in spills, 18.1 against 17.4 ms.)
struct Pixels {
  GlobalF pix, nbr_mean, nbr_var;
  int pitch, nbr_pitch;
  __device__ __forceinline__ explicit Pixels(const ImgDev& im)
      : pix(global(im.pix)), nbr_mean(global(im.nbr_mean)), nbr_var(global(im.nbr_var)), pitch(im.pitch),
        nbr_pitch(im.nbr_pitch) {}
  // count, neighbour mean and neighbour variance at (row, col), 0 where there is no array
  __device__ __forceinline__ void load(int row, int col, float& x, float& mean, float& var) const {
    x = pix[(int64_t)row * pitch + col];
    mean = nbr_mean ? nbr_mean[(int64_t)row * nbr_pitch + col] : 0.f;
    var = nbr_var ? nbr_var[(int64_t)row * nbr_pitch + col] : 0.f;
  }
};

// x in a vector register (a wave-uniform value that would otherwise hold a scalar one across the tile loop).
__device__ __forceinline__ void to_vector(float& x) { asm volatile("" : "+v"(x)); }

// Pixel -> lane layout of a work item, walked by the wavefronts of a block (wave wv takes every WAVES-th
// tile from the wv-th on; the tile, and all state here, is wave-uniform).
//
// Packed (PK, tile width 8): the item's rows as 8-row bands (the image's last band may be shorter),
// each band's pixels in column-major order and the bands back to back; a tile is 64 consecutive
// pixels of that order, an 8 x 8 square except where it wraps from one band into the next, and only
// the item's last tile has dead lanes.  Bands are row_begin + 8 b for a dense item and the kept
// blocks kept[row_begin + b] for a subsampled one.  The walk keeps the tile's band and its place in
// it, so that a lane finds its pixel with one comparison per band of the tile (dividing the pixel's
// index by the band's size, per lane and tile, took 45 vector instructions, five of them quarter-rate
// integer products).
//
// Unpacked (tile width 16, 32 or 64): a grid of tw x (64 / tw) tiles over the item's rows; lanes past
// the image edge are dead.
template <bool PK, int WAVES>
struct TileMap {
  int w, row_lim, n_tiles, t;
  const int* kept;
  int rb;
  // packed: bands, rows of the last band, pixels of a full band and of the item; the tile's band
  // and its first pixel's place in the band
  int nb, hl, bw, npx, b0, q0, first0;
  float inv_hl;
  // unpacked
  int tw_log2, th_log2, tiles_x, q_log2, row_safe;

  __device__ __forceinline__ TileMap(const WorkItem& wi, int w_, int h, int tw_log2_, const int* kept_, int wv) {
    w = w_;
    rb = wi.row_begin;
    kept = kept_;
    row_lim = kept ? h : wi.row_end;
    t = wv;
    nb = kept ? wi.row_end - wi.row_begin : (wi.row_end - wi.row_begin + 7) >> 3;
    if constexpr (PK) {
      hl = min(8, row_lim - band_row(nb - 1));
      bw = w << 3;
      npx = (nb - 1) * bw + hl * w;
      inv_hl = 1.0f / (float)hl;
      n_tiles = (npx + 63) >> 6;
      b0 = 0;
      first0 = band_row(0);
      q0 = wv << 6;
      settle();
    } else {
      tw_log2 = tw_log2_;
      th_log2 = 6 - tw_log2;
      row_safe = kept ? 0 : wi.row_begin;
      tiles_x = (w + (1 << tw_log2) - 1) >> tw_log2;
      q_log2 = 3 - th_log2;
      const int n_rows = kept ? nb << 3 : wi.row_end - wi.row_begin;
      n_tiles = tiles_x * ((n_rows + (1 << th_log2) - 1) >> th_log2);
    }
  }

  __device__ __forceinline__ bool more() const { return t < n_tiles; }
  __device__ __forceinline__ void next() {
    t += WAVES;
    if constexpr (PK) {
      q0 += WAVES << 6;
      settle();
    }
  }
  __device__ __forceinline__ void settle() {
    while (q0 >= bw && b0 < nb - 1) {
      q0 -= bw;
      first0 = band_row(++b0);
    }
  }
  // The tile lies in one band of 8 rows: the common case, whose pixels and box need no per-lane search.
  __device__ __forceinline__ bool plain() const {
    return b0 < nb - 1 ? q0 + 64 <= bw : hl == 8;
  }
  __device__ __forceinline__ int band_row(int b) const { return kept ? kept[rb + b] : rb + (b << 3); }

  // row, column and liveness of this lane's pixel in the tile; dead lanes get an in-image pixel.
  // first: the first row of the pixel's band (packed) or of the tile.
  __device__ __forceinline__ void pixel(int lane, int& row, int& col, bool& live, int& first) const {
    if constexpr (PK) {
      live = (t << 6) + lane < npx;
      int q = q0 + (live ? lane : 0);
      if (plain()) {
        first = first0;
        col = q >> 3;
        row = first0 + (q & 7);
        return;
      }
      int b = b0;
      first = first0;
      for (int k = b0 + 1, lim = bw; k < nb && lim < q0 + 64; ++k, lim += bw) {   // one step where bw >= 64
        const int rk = band_row(k);
        if (q0 + lane >= lim && live) {
          q -= bw;
          b = k;
          first = rk;
        }
      }
      const bool full = b < nb - 1 || hl == 8;
      // q / hl in the last band: (q + 1/2) / hl is at least 1/14 from an integer, so its floor is
      // exact where the quotient's FP32 rounding is below that (at a width of 3e7 it is off by up to 3)
      int cl = (int)(((float)q + 0.5f) * inv_hl);
      if (w > 65536) cl = (int)((unsigned)q / (unsigned)hl);
      col = full ? q >> 3 : cl;
      row = first + (full ? (q & 7) : q - cl * hl);
    } else {
      const int ty = t / tiles_x, tx = t - ty * tiles_x;
      const int row0 = kept ? kept[rb + (ty >> q_log2)] + ((ty & ((1 << q_log2) - 1)) << th_log2)
                            : rb + (ty << th_log2);
      first = row0;
      row = row0 + (lane >> tw_log2);
      col = (tx << tw_log2) + (lane & ((1 << tw_log2) - 1));
      live = row < row_lim && col < w;
      if (!live) {
        row = row_safe;
        col = 0;
      }
    }
  }

  // Box of the tile's live pixels, from this lane's column and band row.  second: a packed tile that
  // runs from the end of one band into the start of the next has a box in each; the first or the
  // second one is returned, and *two says that there is a second.  (A tile spans more than two bands
  // only where a band holds fewer than 64 pixels; its one box is then all columns of its bands.)
  __device__ __forceinline__ TileBox box(int col, int first, bool second, bool* two) const {
    if constexpr (!PK) {
      const int r0 = __builtin_amdgcn_readfirstlane(first);
      const int x0 = (t % tiles_x) << tw_log2;
      *two = false;
      return TileBox{x0, min(w - 1, x0 + (1 << tw_log2) - 1), r0, max(r0, min(row_lim, r0 + (1 << th_log2)) - 1)};
    }
    const int last = min(63, npx - 1 - (t << 6));
    if (plain()) {
      *two = false;
      return TileBox{q0 >> 3, (q0 + last) >> 3, first0, first0 + 7};
    }
    const int c0 = __builtin_amdgcn_readfirstlane(col), s0 = __builtin_amdgcn_readfirstlane(first);
    const int c1 = __builtin_amdgcn_readlane(col, last), s1 = __builtin_amdgcn_readlane(first, last);
    const bool one = s0 == s1, wide = w < 8;
    *two = !one && !wide;
    TileBox b;
    b.x0 = (!one && (wide || second)) ? 0 : c0;
    b.x1 = (one || (second && !wide)) ? c1 : w - 1;
    b.y0 = (*two && second) ? s1 : s0;
    b.y1 = (*two && !second) ? s0 + 7 : min(row_lim, s1 + 8) - 1;
    return b;
  }
};

// The exponent's constants of a component (value path).
struct ValRec {
  float c0, qxx, qxy, qyy;
};

__device__ __forceinline__ ValRec load_val(const float* __restrict__ r) {
  return ValRec{r[tab::R_C0], r[tab::R_QXX], r[tab::R_QXY], r[tab::R_QYY]};
}

// The exponents' constants of N consecutive components in scalar registers, loaded together.
template <int N>
struct ExpoBlock {
  typedef float V4 __attribute__((ext_vector_type(4), aligned(16)));
  V4 v[N];
  __device__ __forceinline__ void load(const float* __restrict__ e) {
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = *reinterpret_cast<const V4*>(e + j * tab::EXPO_REC);
    // used here: sunk to the conditional uses that follow, each would wait for a load of its own
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" ::"s"(v[j]));
  }
  __device__ __forceinline__ ValRec rec(int j) const { return ValRec{v[j].x, v[j].y, v[j].z, v[j].w}; }
};

// acc += density of one component (value path).
__device__ __forceinline__ void comp_value(const ValRec& r, float dxx, float dxy, float dyy, float& acc) {
  acc += ex2(fmaf(r.qxx, dxx, fmaf(r.qxy, dxy, fmaf(r.qyy, dyy, r.c0))));
}

// Which components of an image's galaxy mixture (npsf groups of ncomp, at most 64) can be non-zero on
// a tile.  One component per lane: the lane holds the component's exponent
//   e(d) = c0 - (A dx^2 + B dx dy + C dy^2)   (log2 of its density at offset d)
// and bounds e over the tile's box from above; a component whose bound is below the exact-zero
// threshold is exactly 0 on every pixel of the tile.  The quadratic form is positive definite with
// its minimum at the origin, so its minimum over the box lies on a box edge that faces the origin
// (the segment from any point of the box to the origin leaves the box through such an edge, the
// form falling along it): the nearest edge in x with the best y on it, or the nearest edge in y with
// the best x.  The box's edges are formed by the pixels' own FP32 operations, whose rounding is
// monotonic, so every pixel's computed offset lies in the box; what remains is the rounding of the
// exponents themselves, covered by a slack of 16 ulp of the largest terms on the box plus 0.01.
//
// Against a test of every component's exponent on the tile's pixels (3 FMAs, a compare and a branch
// each) this takes about 30 vector instructions for all components, and the hits are known before
// their records are read, so the next hit's scalar loads are in flight while one is evaluated.
//
// The box says nothing of a component whose constants are not finite or not positive (an estimate's scale or a
// WCS beyond FP32), nor may one be evaluated on pixels where it is 0 if it is so narrow, or so far off, that
// its derivatives' polynomials overflow there (0 times infinity; a PSF of 1e-5 px).  Such a component is odd: it may
// be non-zero on every tile, and a kernel of derivatives then tests it on the tile's pixels (drop_odd).
struct SkipTest {
  float4 form;     // c0, A, B, C; an odd component: infinity, 0, 0, 0
  float4 geo;      // centre offset x, y (the PSF component's), B / 2C, B / 2A
  __device__ __forceinline__ bool odd() const { return form.x == INFINITY; }
};

constexpr float FAR = 1.0e4f;      // offset used by lanes outside the image

// Test of the component with the constants at r, of the PSF component with the star record sr.  reach: the
// largest offset from the source at which its derivatives are formed, 0 where none are.  (With P <= 1.39 times the
// larger of A and C, |P d| stays below 4 * 7e8 and its fourth power below 7e37.)
__device__ __forceinline__ SkipTest skip_test(const float* __restrict__ r, const float* __restrict__ sr, float reach) {
  using namespace tab;
  SkipTest s;
  s.form = make_float4(r[R_C0], -r[R_QXX], -r[R_QXY], -r[R_QYY]);
  const float far = reach + fabsf(sr[S_XIX]) + fabsf(sr[S_XIY]);
  const bool ok = s.form.x < 1e30f && s.form.y >= 0.f && s.form.w >= 0.f && s.form.y * far < 7e8f &&
                  s.form.w * far < 7e8f && fabsf(s.form.z) * far < 1.4e9f;   // false for NaN and infinities
  if (!ok) s.form = make_float4(INFINITY, 0.f, 0.f, 0.f);
  s.geo = make_float4(sr[S_XIX], sr[S_XIY], s.form.w > 0.f ? 0.5f * s.form.z / s.form.w : 0.f,
                      s.form.y > 0.f ? 0.5f * s.form.z / s.form.y : 0.f);
  return s;
}

// ... of galaxy component c
__device__ __forceinline__ SkipTest skip_test_of(const float* __restrict__ T, int c, int ncomp, float reach) {
  using namespace tab;
  return skip_test(T + EXPO + c * EXPO_REC, T + STAR + (c / ncomp) * STAR_REC, reach);
}

// The largest offset from the source on an image's lanes.
__device__ __forceinline__ float reach_of(const ImgDev& im, float psx, float psy) {
  return FAR + (float)max(im.w, im.h) + fabsf(psx) + fabsf(psy);
}

// Upper bound of this lane's component's exponent on the box (psx, psy: the source's position); infinite or NaN
// for an odd component, and NaN where the position is beyond FP32.
__device__ __forceinline__ float exponent_bound(const SkipTest& s, const TileBox& b, float psx, float psy) {
  const float xl = ((float)b.x0 - psx) - s.geo.x, xh = ((float)b.x1 - psx) - s.geo.x;
  const float yl = ((float)b.y0 - psy) - s.geo.y, yh = ((float)b.y1 - psy) - s.geo.y;
  const float A = s.form.y, B = s.form.z, C = s.form.w;
  const float xn = __builtin_amdgcn_fmed3f(xl, 0.f, xh), yn = __builtin_amdgcn_fmed3f(yl, 0.f, yh);
  const float ys = __builtin_amdgcn_fmed3f(-s.geo.z * xn, yl, yh);
  const float xs = __builtin_amdgcn_fmed3f(-s.geo.w * yn, xl, xh);
  const float q1 = fmaf(A * xn, xn, ys * fmaf(B, xn, C * ys));
  const float q2 = fmaf(C * yn, yn, xs * fmaf(B, yn, A * xs));
  const float X = fmaxf(fabsf(xl), fabsf(xh)), Y = fmaxf(fabsf(yl), fabsf(yh));
  const float M = fmaf(X, fmaf(A, X, fabsf(B) * Y), C * Y * Y);
  return (s.form.x - fminf(q1, q2)) + fmaf(M, 0x1p-20f, 0.01f);
}

// True on the lanes whose component must be evaluated on the box: one that may be non-zero, or NaN.
__device__ __forceinline__ bool may_hit(const SkipTest& s, const TileBox& b, float psx, float psy, float e_zero) {
  return !(exponent_bound(s, b, psx, psy) < e_zero);
}

// Brings an image's whole table (n floats) into the cache behind the scalar loads that will read it,
// 128 bytes per lane of the block's second wavefront, while the first one forms the skip tests.  The
// tables of a large batch come from HBM, and a record's first scalar load would wait for it hit by hit.
__device__ __forceinline__ void touch_table(const float* __restrict__ T, int n) {
  for (int i = ((int)threadIdx.x - 64) * 32; i >= 0 && i < n; i += 64 * 32) {
    const float v = T[i];
    asm volatile("" ::"v"(v));
  }
}

// Index of the lowest set bit of m, or 64 if there is none.
__device__ __forceinline__ int low_bit(unsigned long long m) { return m ? __builtin_ctzll(m) : 64; }

// The lanes below n (n <= 64).
__device__ __forceinline__ unsigned long long lane_mask(int n) { return n >= 64 ? ~0ull : (1ull << n) - 1; }

// Components (bit = the lane holding the component's test) that must be evaluated on tm's tile; col and
// first are this lane's from tm.pixel.
template <class MAP>
__device__ __forceinline__ unsigned long long tile_hits(const SkipTest& s, const MAP& tm, int col, int first,
                                                        float psx, float psy, float e_zero) {
  bool two;
  unsigned long long hits = __ballot(may_hit(s, tm.box(col, first, false, &two), psx, psy, e_zero));
  if (two) hits |= __ballot(may_hit(s, tm.box(col, first, true, &two), psx, psy, e_zero));
  return hits;
}

// The threshold of a work item of the derivative kernels, with its last bit set where the item has an odd component (lanes:
// the components' lanes).  A mark in a scalar that the tile loop holds anyway: one more of them, or a vector
// comparison a tile, cost the value+gradient+Hessian kernel 2%.
__device__ __forceinline__ float mark_odd(float e_zero, const SkipTest& s, unsigned long long lanes) {
  const bool odd = (__ballot(s.odd()) & lanes) != 0ull;
  // slightly lower, which skips no more; -infinity becomes the lowest finite value
  return odd ? __uint_as_float(e_zero == -INFINITY ? 0xff7fffffu : __float_as_uint(e_zero) | 1u) : e_zero;
}

// hits without the odd components whose exponent reaches the threshold on no pixel of the tile (dx0, dy0: this
// lane's offset from the source); where e_zero bears no mark, hits.
__device__ __forceinline__ unsigned long long drop_odd(unsigned long long hits, const SkipTest& s,
                                                       const float* __restrict__ T, int ncomp, float dx0, float dy0,
                                                       float e_zero) {
  using namespace tab;
  if (__builtin_expect(__float_as_uint(e_zero) & 1u, 0)) {
    for (unsigned long long odd = __ballot(s.odd()) & hits; odd; odd &= odd - 1) {
      const int c = __builtin_ctzll(odd);
      const float* __restrict__ sr = T + STAR + (c / ncomp) * STAR_REC;
      const ValRec r = load_val(T + EXPO + c * EXPO_REC);
      const float dx = dx0 - sr[S_XIX], dy = dy0 - sr[S_XIY];
      const float e = fmaf(r.qxx, dx * dx, fmaf(r.qxy, dx * dy, fmaf(r.qyy, dy * dy, r.c0)));
      if (!__ballot(e >= e_zero)) hits &= ~(1ull << c);
    }
  }
  return hits;
}

}  // namespace
}  // namespace celeste
