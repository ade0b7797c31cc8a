// Surrogate initialiser network: hand-written training and inference kernels.
//
// A small CNN maps a source's 5-band 32x32 patch to its 27 parameters (in
// standardised unconstrained coordinates) so that the trust-region fit starts
// closer to the optimum; the plain start remains the fallback.  Layers: four
// 3x3 same convolutions (5->32->64->64->128, ReLU, 2x2 max-pool after the last
// three) and dense 2048->256 (ReLU) -> 27.  Every matrix product runs on the BF16 matrix
// cores (16x16x32 MFMA, FP32 accumulation): the convolutions' forward and data-gradient products on
// kernels that stage an image's pixels once for all taps (k_conv1, k_conv3: bias, ReLU, pooling and the
// sum of K splits in them), their weight gradients and the dense layers on a
// gather-GEMM (k_gemm, split-K partials summed in a fixed order).  Activations and
// gradients feeding a product are BF16; master weights, Adam moments, biases and
// all reductions are FP32.
#include <math.h>

#include <algorithm>
#include <cstdint>
#include <cmath>
#include <new>
#include <string>

#include "celeste_internal.h"
#include "wave.h"

namespace celeste {

typedef __bf16 bf16;

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ __forceinline__ bf16 to_bf16(float x) { return (bf16)x; }
__device__ __forceinline__ float from_bf16(bf16 x) { return (float)x; }

constexpr int TM = 64, TN = 64, TK = 32, TKP = TK + 8;

// ------------------------------------------------------------------ gather loaders
// A loader gives 8 consecutive k of A(m, k) (a8), zero for k >= kend or an index out of range.
// For B(k, n) it gives either 8 consecutive k at one n (b8; kRunN false) or 8 consecutive n at one k
// (b8n; kRunN true), n a multiple of 8.
// Likewise for A: 8 consecutive k at one m (a8; kRunM false) or 8 consecutive m at one k (a8m; kRunM
// true).  An operand stored with its other index running is read in runs of that one: 16-byte loads
// where element loads along k would touch a line each (256 x 2048 weight gradient over 256 images:
// 33 us by elements, 10 us by runs).

// kk -> (ky, kx) of a 3x3 kernel tap
__device__ __forceinline__ int tap_y(int kk) { return (kk * 11) >> 5; }   // kk / 3 for kk < 9
__device__ __forceinline__ int tap_x(int kk) { return kk - 3 * tap_y(kk); }

__device__ __forceinline__ bf16x8_t zero8() {
  bf16x8_t z;
#pragma unroll
  for (int j = 0; j < 8; ++j) z[j] = (bf16)0.f;
  return z;
}

// 8 contiguous BF16 values at p: one 16-byte load where p is aligned and all 8 are wanted, else
// element by element (the first n_valid).
__device__ __forceinline__ bf16x8_t load8(const bf16* p, int n_valid, bool aligned) {
  if (n_valid >= 8 && aligned && ((uintptr_t)p & 15) == 0) return *reinterpret_cast<const bf16x8_t*>(p);
  bf16x8_t v = zero8();
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (j < n_valid) v[j] = p[j];
  return v;
}

// The 8 pixels px + sh .. px + sh + 7 of one image row (zero outside 0 .. wd-1), px a multiple of 8,
// sh in {-1, 0, 1}, row 16-byte aligned: the aligned 16 bytes at px and, for sh = -1 (+1), the 16 bytes
// before (after) them, shifted by one element with funnel shifts; a neighbour chunk outside the row
// reads as zeros.
__device__ __forceinline__ bf16x8_t row8(const bf16* __restrict__ row, int px, int sh, int wd) {
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
  const u32x4_t zero = {0u, 0u, 0u, 0u};
  const u32x4_t mid = *reinterpret_cast<const u32x4_t*>(row + px);
  const u32x4_t lo = (sh < 0 && px > 0) ? *reinterpret_cast<const u32x4_t*>(row + px - 8) : zero;
  const u32x4_t hi = (sh > 0 && px + 8 < wd) ? *reinterpret_cast<const u32x4_t*>(row + px + 8) : zero;
  // window w = {lo.w, mid.x, mid.y, mid.z, mid.w, hi.x}; output dword i = (w[i+1+up] : w[i+up]) >> bits
  const unsigned w[6] = {lo.w, mid.x, mid.y, mid.z, mid.w, hi.x};
  const unsigned bits = sh == 0 ? 0u : 16u;
  const int up = sh < 0 ? 0 : 1;
  u32x4_t o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned a = up ? w[i + 2] : w[i + 1], b = up ? w[i + 1] : w[i];
    o[i] = __builtin_amdgcn_alignbit(a, b, bits);
  }
  return __builtin_bit_cast(bf16x8_t, o);
}

struct LdConvWgrad {      // dW[co][ci*9+kk] = sum_{img,p} dY[img][co][p] X[img][ci][p + off(kk)]
  static constexpr bool kRunN = false;
  static constexpr bool kRunM = false;
  const bf16* dY;
  const bf16* X;
  int Cin, Cout, hwl, wl;   // image side 2^wl, HW = 2^hwl
  // k = img*HW + p; HW, the K splits and the run's first k are multiples of 8, so a run is whole
  // and stays in one image row (the image side is a power of two of at least 8)
  __device__ bf16x8_t a8(int m, int k, int kend) const {
    const int img = k >> hwl, p = k & ((1 << hwl) - 1);
    return load8(dY + ((((size_t)img * Cout + m) << hwl) + p), kend - k, true);
  }
  __device__ bf16x8_t b8(int k, int n, int) const {
    const int img = k >> hwl, p = k & ((1 << hwl) - 1), py = p >> wl, px = p & ((1 << wl) - 1);
    const int ci = n / 9, kk = n - ci * 9;
    const int y = py + tap_y(kk) - 1;
    if (y < 0 || y >= (1 << wl)) return zero8();
    return row8(X + ((((size_t)img * Cin + ci) << hwl) + ((size_t)y << wl)), px, tap_x(kk) - 1, 1 << wl);
  }
};

struct LdFcFwd {          // Y[o][b] = sum_i W[o][i] X[b][i]
  static constexpr bool kRunN = false;
  static constexpr bool kRunM = false;
  const bf16* W;
  const bf16* X;
  int In;
  __device__ bf16x8_t a8(int m, int k, int kend) const {
    return load8(W + (size_t)m * In + k, kend - k, (In & 7) == 0);
  }
  __device__ bf16x8_t b8(int k, int n, int kend) const {
    return load8(X + (size_t)n * In + k, kend - k, (In & 7) == 0);
  }
};

struct LdFcDgrad {        // dX[i][b] = sum_o W[o][i] dY[b][o]
  static constexpr bool kRunN = false;
  static constexpr bool kRunM = true;
  const bf16* W;
  const bf16* dY;
  int In, Out;
  __device__ bf16x8_t a8m(int m, int k, int M) const {
    return load8(W + (size_t)k * In + m, M - m, (In & 7) == 0);
  }
  __device__ bf16x8_t b8(int k, int n, int kend) const {
    return load8(dY + (size_t)n * Out + k, kend - k, ((size_t)n * Out + k) % 8 == 0);
  }
};

struct LdFcWgrad {        // dW[o][i] = sum_b dY[b][o] X[b][i]
  static constexpr bool kRunN = true;
  static constexpr bool kRunM = true;
  const bf16* dY;
  const bf16* X;
  int In, Out;            // In a multiple of 8
  __device__ bf16x8_t a8m(int m, int k, int M) const {
    return load8(dY + (size_t)k * Out + m, M - m, (Out & 7) == 0);
  }
  __device__ bf16x8_t b8n(int k, int n) const { return load8(X + (size_t)k * In + n, 8, true); }
};

// C[z][m][n] = sum over the z-th K split of A(m,k) B(k,n).  Block 256 = 4 waves in a 2x2
// arrangement over a 64 x 64 tile, each wave a 32 x 32 sub-tile of 2 x 2 MFMA
// 16x16x32 tiles.  Operand runs of 8 BF16 go to LDS (k-runs as 16-byte stores, m- and n-runs
// transposed element by element) and come back as single 16-byte reads; the next K step's
// operands are loaded into registers while the current step's products run.
template <class LD>
__global__ __launch_bounds__(256) void k_gemm(LD ld, int M, int N, int K, int kchunk, float* __restrict__ C) {
  constexpr int NJ = TN / 32;
  __shared__ __align__(16) bf16 As[TM][TKP];
  __shared__ __align__(16) bf16 Bs[TN][TKP];
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
  const int kbeg = blockIdx.z * kchunk, kend = min(K, kbeg + kchunk);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int wm = (wv >> 1) * 32, wn = (wv & 1) * (TN / 2);
  f32x4_t acc[2][NJ];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // k-runs: row t / 4, k-run (t % 4) * 8.  m- and n-runs: k = t % 32, rows 8 (t / 32) .. + 7 (the 32
  // lanes of one run write 32 consecutive k of an LDS row, so the transposed stores spread over the banks).
  const int ar = t >> 2, ak = (t & 3) * 8;
  const int nb = 8 * (t >> 5), kb = t & 31;
  bf16x8_t an, bn;
  auto fetch = [&](int k0) {
    if constexpr (LD::kRunM) {
      const int m = m0 + nb, k = k0 + kb;
      an = (m < M && k < kend) ? ld.a8m(m, k, M) : zero8();
    } else {
      const int m = m0 + ar, k = k0 + ak;
      an = (m < M && k < kend) ? ld.a8(m, k, kend) : zero8();
    }
    if constexpr (LD::kRunN) {
      const int n = n0 + nb, k = k0 + kb;
      bn = (n < N && k < kend) ? ld.b8n(k, n) : zero8();
    } else {
      const int n = n0 + ar, k = k0 + ak;
      bn = (n < N && k < kend) ? ld.b8(k, n, kend) : zero8();
    }
  };
  bf16x8_t a[2], b[NJ];
  fetch(kbeg);
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  for (int k0 = kbeg; k0 < kend; k0 += TK) {
    if constexpr (LD::kRunM) {
#pragma unroll
      for (int j = 0; j < 8; ++j) As[nb + j][kb] = an[j];
    } else {
      *reinterpret_cast<bf16x8_t*>(&As[ar][ak]) = an;
    }
    if constexpr (LD::kRunN) {
#pragma unroll
      for (int j = 0; j < 8; ++j) Bs[nb + j][kb] = bn[j];
    } else {
      *reinterpret_cast<bf16x8_t*>(&Bs[ar][ak]) = bn;
    }
    __syncthreads();
    if (k0 + TK < kend) fetch(k0 + TK);   // next step's operands, in flight during the products
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8_t*>(&As[wm + i * 16 + r16][kq]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[j] = *reinterpret_cast<const bf16x8_t*>(&Bs[wn + j * 16 + r16][kq]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  }
  float* Cz = C + (size_t)blockIdx.z * M * N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mm = m0 + wm + i * 16 + (lane >> 4) * 4 + r;
        const int nn = n0 + wn + j * 16 + (lane & 15);
        if (mm < M && nn < N) Cz[(size_t)mm * N + nn] = acc[i][j][r];
      }
}

// ------------------------------------------------------------------ convolutions
// The convolution kernels' wavefronts work on 16-pixel fragments of 2 rows x 8 pixels, whole pooling windows; after
// the products lane (px = lane & 15, kq = lane >> 4) holds channels 4 kq .. 4 kq + 3 of the fragment's px-th pixel.
// Storing those one value at a time (64 two-byte stores per 64 x 64 outputs) took longer than the
// products; here a quad of lanes exchanges its 4 channels x 4 pixels first.
struct FragStore {
  int px;
  unsigned sel0, sel1;
  __device__ __forceinline__ explicit FragStore(int px_) : px(px_) {
    constexpr unsigned kLo = 0x05040100u, kHi = 0x07060302u, kLoR = 0x01000504u, kHiR = 0x03020706u;
    sel0 = px & 2 ? (px & 1 ? kHiR : kHi) : (px & 1 ? kLoR : kLo);
    sel1 = px & 2 ? (px & 1 ? kLoR : kLo) : (px & 1 ? kHiR : kHi);
  }
  // bf16(relu(v + b)) of the four channels; this lane stores channel px & 3 of its quad's 4 pixels at dst
  __device__ __forceinline__ void act(const f32x4_t& v, const f32x4_t& b, bf16* dst) const {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
    unsigned w[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
      w[h] = __builtin_bit_cast(unsigned, bf16x2_t{to_bf16(fmaxf(v[2 * h] + b[2 * h], 0.f)),
                                                   to_bf16(fmaxf(v[2 * h + 1] + b[2 * h + 1], 0.f))});
    const bool b1 = px & 2, b0 = px & 1;
    const unsigned keep = b1 ? w[1] : w[0], got2 = dpp_u<DPP_XOR2>(b1 ? w[0] : w[1]);   // 2 channels, pixels px, px ^ 2
    const unsigned lo = __builtin_amdgcn_perm(got2, keep, 0x05040100u), hi = __builtin_amdgcn_perm(got2, keep, 0x07060302u);
    const unsigned mine = b0 ? hi : lo, got1 = dpp_u<DPP_XOR1>(b0 ? lo : hi);           // 1 channel, px ^ 1, px ^ 3
    const uint2 o = make_uint2(__builtin_amdgcn_perm(got1, mine, sel0), __builtin_amdgcn_perm(got1, mine, sel1));
    *reinterpret_cast<uint2*>(dst) = o;
  }
  // the channel of four whose pooled value this lane stores
  __device__ __forceinline__ int pool_channel() const { return (px & 1) + ((px >> 2) & 2); }
  // 2x2 max-pool of bf16(relu(v + b)): relu, the addition and the rounding keep order, so the largest v is taken first.
  // This lane stores its window's value of pool_channel(), whose bias is bc, at dst.
  __device__ __forceinline__ void pool(const f32x4_t& v, float bc, bf16* dst) const {
    float m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m[r] = fmaxf(v[r], dpp<DPP_XOR1>(v[r]));
      m[r] = fmaxf(m[r], dpp<DPP_XOR8>(m[r]));
    }
    const float a = px & 1 ? m[1] : m[0], c = px & 1 ? m[3] : m[2];
    *dst = to_bf16(fmaxf((px & 8 ? c : a) + bc, 0.f));
  }
  template <int CTRL>
  static __device__ __forceinline__ unsigned dpp_u(unsigned x) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
  }
};

// First convolution: 5 channels of 32 x 32 images to 32, k = ci*9+kk (45, two 32-deep steps), act = bf16(relu(. + bias)).
// A block takes 8 rows of an image, 64 pixels a wavefront; the image's rows and border are staged as they lie and
// a lane gathers its 8 k of a step by per-lane offsets, fixed over the fragments.  Bound by the activation it
// writes (64 KB an image): 4,000 images 100 us (365 us as a gather-GEMM with a transposing LDS
// store per element and half its rows unused).
constexpr int C1_IN = 5, C1_OUT = 32, C1_K = 45;
__global__ __launch_bounds__(256) void k_conv1(const bf16* __restrict__ wfrag, const bf16* __restrict__ X,
                                               const float* __restrict__ bias, bf16* __restrict__ act) {
  constexpr int W = 32, R = 8, LP = 48, X0 = 8;   // LDS row pitch; column of pixel 0 (16-byte aligned)
  constexpr int NF = 4, MF = C1_OUT / 16;
  __shared__ __align__(16) bf16 lds[C1_IN][R + 2][LP];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int img = blockIdx.x >> 2, y0 = (blockIdx.x & 3) * R;
  for (int i = t; i < C1_IN * (R + 2) * (LP / 8); i += 256) {
    const int x8 = i % (LP / 8), row = i / (LP / 8), ci = row / (R + 2), r = row - ci * (R + 2), y = y0 + r - 1;
    const bool in = x8 >= 1 && x8 <= W / 8 && y >= 0 && y < W;
    *reinterpret_cast<bf16x8_t*>(&lds[ci][r][8 * x8]) =
        in ? *reinterpret_cast<const bf16x8_t*>(X + ((((size_t)img * C1_IN + ci) * W + y) * W + 8 * (x8 - 1))) : zero8();
  }
  const int px = lane & 15, kq = lane >> 4;
  bf16x8_t a[2][MF];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < MF; ++i) a[s][i] = *reinterpret_cast<const bf16x8_t*>(wfrag + ((s * MF + i) * 64 + lane) * 8);
  int off[2][8];      // element offset of k from the pixel's own place
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = min(s * 32 + kq * 8 + j, C1_K - 1), ci = k / 9, kk = k - ci * 9;
      off[s][j] = ci * ((R + 2) * LP) + tap_y(kk) * LP + tap_x(kk) - 1;
    }
  const FragStore st(px);
  f32x4_t b4[MF];
#pragma unroll
  for (int i = 0; i < MF; ++i) b4[i] = *reinterpret_cast<const f32x4_t*>(bias + 16 * i + 4 * kq);
  __syncthreads();
  const bf16* flat = &lds[0][0][0];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int g = wv * NF + f, y = 2 * (g >> 2) + (px >> 3), x = 8 * (g & 3) + (px & 7);
    const bf16* at = flat + y * LP + X0 + x;
    bf16x8_t b[2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bf16 v = at[off[s][j]];
        b[s][j] = s == 0 || 32 + kq * 8 + j < C1_K ? v : (bf16)0.f;
      }
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      f32x4_t acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[0], f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][i], b[1], acc, 0, 0, 0);
      const int m = 16 * i + 4 * kq + (px & 3);
      st.act(acc, b4[i], act + (((size_t)img * C1_OUT + m) * W + y0 + y) * W + (x & ~3));
    }
  }
}

// 3x3 same convolution of images of side 2^WL with 2^CL channels (layers 1 .. 3), forward and data gradient
// (FLIP: the taps mirrored), as an implicit product over k = tap * 2^CL + channel in 32-deep steps.
// A block of four wavefronts takes 64 NF pixels (rows of one image, or whole images) of 16 MF output channels.  It
// stages every channel of its pixels and their border once, pixel-major with a zero border, so that the operand of
// each tap is the same LDS data at a constant offset: the K loop has neither barriers nor addresses,
// only the weights' fragments (k_conv_weights) to load from cache.  A wavefront's 16-pixel
// fragments are 2 rows x 8 pixels, whole pooling windows, so the pooled image is formed from the
// accumulators.  LDS pitch: 16 bytes more than a pixel's channels, 4 banks apart modulo 32, so that the
// 16-byte reads of 8 neighbouring pixels do not collide.
// Sums stay those of the K splits that the layer's size asks for (chunk: steps of one split), added in order.
// Bound by the matrix cores and the LDS reads that feed them (16 MF NF products' operands come
// from MF + NF reads).  4,000 images, the three forward products with pooling: 438 us; 256 images,
// data gradients: 20 us each.  (Gathering each tap's operand anew, transposed through LDS element by
// element with two barriers a step: 1,110 us and 224 us more for the pooling; 37 us each.)
template <int CL, int WL, int MF, int NF, bool FLIP>
__global__ __launch_bounds__(256) void k_conv3(const bf16* __restrict__ wfrag, const bf16* __restrict__ X, int B, int M,
                                               int chunk, const float* __restrict__ bias, bf16* __restrict__ act,
                                               bf16* __restrict__ pool, float* __restrict__ out) {
  constexpr int CH = 1 << CL, W = 1 << WL, NPX = 64 * NF;
  constexpr int R = W * W < NPX ? W : NPX / W, NI = NPX / (R * W);   // rows of an image, images
  constexpr int WP = W + 2, RP = R + 2, PB = CH * 2 + 16;            // with border; bytes per pixel
  __shared__ __align__(16) unsigned char lds[NI * RP * WP * PB];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int first = (int)blockIdx.x * (NPX / 64);        // in runs of 64 pixels
  const int img0 = first >> (2 * WL - 6), y0 = ((first & ((1 << (2 * WL - 6)) - 1)) << 6) >> WL;
  // ---- stage: 4 channels x 8 pixels per thread and turn, channels fastest over the lanes
  constexpr int CG = CH / 4, XG = W / 8, ROWS = NI * RP;
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
  for (int i = t; i < ROWS * XG * CG; i += 256) {
    const int cg = i & (CG - 1), x8 = (i / CG) & (XG - 1), row = i / (CG * XG);
    const int ni = row / RP, y = y0 + (row - ni * RP) - 1;
    bf16x8_t v[4];
    const bool in = y >= 0 && y < W && img0 + ni < B;
    const bf16* src = X + ((((size_t)(img0 + ni) * CH + 4 * cg) << (2 * WL)) + ((size_t)(in ? y : 0) << WL) + 8 * x8);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = in ? *reinterpret_cast<const bf16x8_t*>(src + ((size_t)c << (2 * WL))) : zero8();
    unsigned char* dst = lds + (row * WP + 1 + 8 * x8) * PB + cg * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) *reinterpret_cast<bf16x4_t*>(dst + j * PB) = bf16x4_t{v[0][j], v[1][j], v[2][j], v[3][j]};
  }
  constexpr int CV = CH / 8;
  for (int i = t; i < ROWS * 2 * CV; i += 256) {
    const int c = i & (CV - 1), side = (i / CV) & 1, row = i / (2 * CV);
    *reinterpret_cast<bf16x8_t*>(lds + (row * WP + side * (W + 1)) * PB + c * 16) = zero8();
  }
  __syncthreads();
  // ---- products
  const int px = lane & 15, kq = lane >> 4;
  int at[NF];         // LDS byte of this lane's pixel of each fragment, at the first tap
  int py[NF], pi[NF], pxx[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int g = wv * NF + f, x8 = g & (XG - 1), r2 = 2 * (g / XG), ni = r2 / R, r = r2 - ni * R;
    py[f] = r + (px >> 3);
    pxx[f] = 8 * x8 + (px & 7);
    pi[f] = ni;
    at[f] = ((ni * RP + py[f]) * WP + pxx[f]) * PB + kq * 16;
  }
  const int m16 = M >> 4, mb0 = blockIdx.y * MF;
  const bf16* wl = wfrag + ((size_t)mb0 * 64 + lane) * 8;
  constexpr int CB = CH / 32, STEPS = 9 * CB;
  f32x4_t acc[MF][NF], sum[MF][NF];
#pragma unroll
  for (int i = 0; i < MF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (NF < 4) sum[i][j] = f32x4_t{-0.f, -0.f, -0.f, -0.f};   // -0 + x is x
    }
  bf16x8_t a[2][MF];
  auto weights = [&](int step, bf16x8_t (&d)[MF]) {
#pragma unroll
    for (int i = 0; i < MF; ++i) d[i] = *reinterpret_cast<const bf16x8_t*>(wl + ((size_t)step * m16 + i) * 512);
  };
  weights(0, a[0]);
  int left = chunk;
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int kk = s / CB, ty = FLIP ? 2 - kk / 3 : kk / 3, tx = FLIP ? 2 - kk % 3 : kk % 3;
    const int tap = (ty * WP + tx) * PB + (s % CB) * 64;
    bf16x8_t b[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) b[j] = *reinterpret_cast<const bf16x8_t*>(lds + at[j] + tap);
    if (s + 1 < STEPS) weights(s + 1, a[(s + 1) & 1]);
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s & 1][i], b[j], acc[i][j], 0, 0, 0);
    if constexpr (NF < 4) {
      if (--left == 0 || s + 1 == STEPS) {   // the end of a split
        left = chunk;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
          for (int j = 0; j < NF; ++j) {
            sum[i][j] += acc[i][j];
            acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  }
  // ---- results
  const FragStore st(px);
  f32x4_t b4[MF];
  float bc[MF];
#pragma unroll
  for (int i = 0; i < MF; ++i)
    if constexpr (!FLIP) {
      const float* bm = bias + (mb0 + i) * 16 + 4 * kq;
      b4[i] = *reinterpret_cast<const f32x4_t*>(bm);
      bc[i] = bm[st.pool_channel()];
    }
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const int img = img0 + pi[j];
    if (img >= B) continue;   // the same on the lanes of a fragment
    const int y = y0 + py[j], x = pxx[j];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      f32x4_t v;
      if constexpr (NF < 4) v = sum[i][j]; else v = acc[i][j];
      const int m = (mb0 + i) * 16 + 4 * kq;
      if constexpr (FLIP) {
#pragma unroll
        for (int r = 0; r < 4; ++r) out[((size_t)(m + r) * B + img) * (W * W) + y * W + x] = v[r];
      } else {
        const size_t plane = (size_t)img * M + m;
        if (act) st.act(v, b4[i], act + ((plane + (px & 3)) << (2 * WL)) + y * W + (x & ~3));
        st.pool(v, bc[i], pool + ((plane + st.pool_channel()) << (2 * WL - 2)) + (y >> 1) * (W / 2) + (x >> 1));
      }
    }
  }
}

// Sum over the K splits in split order; 8 loads in flight at a time.
__device__ __forceinline__ float split_sum(const float* C, int S, size_t MN, size_t idx) {
  float s = C[idx];
  int z = 1;
  for (; z + 8 <= S; z += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = C[(size_t)(z + j) * MN + idx];
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; z < S; ++z) s += C[(size_t)z * MN + idx];
  return s;
}

// ------------------------------------------------------------------ epilogues and elementwise

// The elementwise passes over images work on units of 2 rows x 8 columns of one channel of one image (image
// side 2^wl >= 8): 16-byte loads and stores, four whole pooling windows, and shifts instead of divisions by
// the image's shape.
struct Unit {
  size_t plane;   // first element of the channel's image
  int p, q;       // the unit's first pixel in it, and in the pooled image
};
__device__ __forceinline__ Unit unit_at(size_t plane_index, int u, int wl) {
  const int y2 = u >> (wl - 3), x8 = u & ((1 << (wl - 3)) - 1);
  return Unit{plane_index << (2 * wl), (y2 << (wl + 1)) + 8 * x8, (y2 << (wl - 1)) + 4 * x8};
}

__device__ __forceinline__ bf16x8_t ld8(const bf16* p) { return *reinterpret_cast<const bf16x8_t*>(p); }
__device__ __forceinline__ void st8(bf16* p, const bf16x8_t& v) { *reinterpret_cast<bf16x8_t*>(p) = v; }

// dense forward: out[b][o] = C[o][b] + bias[o], ReLU + BF16 (hidden) or FP32 (output)
__global__ void k_ep_fc_fwd(const float* __restrict__ C, int S, int Out, int B, const float* __restrict__ bias,
                            bf16* __restrict__ act, float* __restrict__ outf) {
  const int total = Out * B;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int o = i % Out, b = i / Out;
    const float v = split_sum(C, S, (size_t)Out * B, (size_t)o * B + b) + bias[o];
    if (act) act[i] = to_bf16(fmaxf(v, 0.f));
    if (outf) outf[i] = v;
  }
}

// Convolution weight gradient dW[m][n] = sum_z C[z][m][n] over S splits, in order, and, in the last blocks, a
// bias gradient per thread from its channel's slices.  The smallest layer has 1,440 entries and up to
// 1,024 splits, so its time is the chain of loads: a block takes 32 consecutive entries, all its threads load
// (128 splits at a time, the next ones in flight) and one per entry adds, from LDS.  256 images, mean of the
// four layers: 7.4 us (a thread per entry, 8 loads in flight, and a launch for the biases: 14.1 and 4.5 us).
constexpr int BP_PARTS = 64;   // slices of a channel's bias gradient
constexpr int GS_COLS = 32, GS_GROUPS = 8, GS_DEPTH = 16;
__global__ __launch_bounds__(256) void k_grad_sum(const float* __restrict__ C, int S, int MN, int n_blocks_w,
                                                  float* __restrict__ gw, const float* __restrict__ bpart, int Cch,
                                                  float* __restrict__ gb) {
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= n_blocks_w) {
    const int c = ((int)blockIdx.x - n_blocks_w) * 256 + t;
    if (c >= Cch) return;
    float s = 0.f;
#pragma unroll 16
    for (int q = 0; q < BP_PARTS; ++q) s += bpart[c * BP_PARTS + q];
    gb[c] = s;
    return;
  }
  constexpr int STEP = GS_GROUPS * GS_DEPTH;
  __shared__ float sh[2][STEP][GS_COLS];
  const int col = t & (GS_COLS - 1), g = t / GS_COLS, idx = (int)blockIdx.x * GS_COLS + col;
  const float* src = C + min(idx, MN - 1);
  float v[GS_DEPTH], s = -0.f;   // -0 + x is x
  auto fetch = [&](int z0) {
#pragma unroll
    for (int k = 0; k < GS_DEPTH; ++k) v[k] = src[(size_t)min(z0 + g + GS_GROUPS * k, S - 1) * MN];
  };
  fetch(0);
  for (int z0 = 0, b = 0; z0 < S; z0 += STEP, b ^= 1) {
#pragma unroll
    for (int k = 0; k < GS_DEPTH; ++k) sh[b][g + GS_GROUPS * k][col] = v[k];
    __syncthreads();   // one a step: the other buffer is written only after every sum over it
    if (z0 + STEP < S) fetch(z0 + STEP);
    if (g == 0) {
      const int n = min(STEP, S - z0);
      int k = 0;
      for (; k + 16 <= n; k += 16) {
        float w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = sh[b][k + j][col];
#pragma unroll
        for (int j = 0; j < 16; ++j) s += w[j];
      }
      for (; k < n; ++k) s += sh[b][k][col];
    }
  }
  if (g == 0 && idx < MN) gw[idx] = s;
}

// Backward through (optional) 2x2 max-pool and ReLU.  g comes from a GEMM as C[c*Hg*Wg + q][img]
// (DENSE, summed over splits) or C[c][img*Hg*Wg + q] (convolution); r is the post-ReLU
// activation at full resolution (side 2^wl).  The pooled gradient goes to the first maximal
// input of its window (row-major), then is masked by r > 0.  A wavefront takes the q-th of BP_PARTS
// slices of a channel's pixels (over images and positions) in runs of 1,024, a unit per lane, and
// sums the FP32 gradient over the slice for the bias: 256 strided sums, then a tree.
// Bound by memory: the gradient and the activation read, the BF16 result written.  256 images, mean of the four
// layers: 14 us (39 us with an element per thread, its FP32 gradient written for a pass of 12 us over it).
constexpr int PRB_RUN = 1024;

template <bool POOLED, bool DENSE>
__device__ __forceinline__ void pool_relu_unit(const float* __restrict__ C, int S, int B, size_t MN, int c, int img,
                                               int gl, int wl, const Unit& u, const bf16x8_t& a0, const bf16x8_t& a1,
                                               float (&d)[2][8]) {
  if constexpr (POOLED) {
    f32x4_t g;
    if constexpr (DENSE) {
#pragma unroll
      for (int j = 0; j < 4; ++j) g[j] = split_sum(C, S, MN, ((((size_t)c << gl) + u.q + j)) * B + img);
    } else {
      g = *reinterpret_cast<const f32x4_t*>(C + (((size_t)c * B + img) << gl) + u.q);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v[4] = {from_bf16(a0[2 * j]), from_bf16(a0[2 * j + 1]), from_bf16(a1[2 * j]),
                          from_bf16(a1[2 * j + 1])};
      const float mx = fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
      const int first = v[0] == mx ? 0 : v[1] == mx ? 1 : v[2] == mx ? 2 : 3;
#pragma unroll
      for (int m = 0; m < 4; ++m) d[m >> 1][2 * j + (m & 1)] = (first == m && v[m] > 0.f) ? g[j] : 0.f;
    }
  } else {
    static_assert(!DENSE, "the dense layer follows a pooled one");
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4_t g = *reinterpret_cast<const f32x4_t*>(C + (((size_t)c * B + img) << gl) + u.p + (y << wl) + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) d[y][4 * h + j] = from_bf16((y ? a1 : a0)[4 * h + j]) > 0.f ? g[j] : 0.f;
      }
  }
}

template <bool POOLED, bool DENSE>
__global__ __launch_bounds__(256) void k_pool_relu_bwd(const float* __restrict__ C, int S, int B, int Cch, int wl,
                                                       const bf16* __restrict__ r, bf16* __restrict__ dzb,
                                                       float* __restrict__ bpart) {
  __shared__ float run[4][PRB_RUN];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = blockIdx.y, slice = (int)blockIdx.x * 4 + wv;
  const int gl = POOLED ? 2 * wl - 2 : 2 * wl, xl = wl - 3;   // 2^xl units per pair of rows
  const size_t MN = ((size_t)Cch * B) << gl;
  const int n = B << (2 * wl), per = (n + BP_PARTS - 1) / BP_PARTS;
  const int i0 = min(n, slice * per), i1 = min(n, i0 + per);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};   // strided sums lane, lane + 64, + 128, + 192
  for (int a = i0; a < i1; a += PRB_RUN) {
    const int b = min(i1, a + PRB_RUN);   // pixels [a, b): units of the row pairs they lie in
    const int u0 = (a >> (wl + 1)) << xl, u1 = (((b - 1) >> (wl + 1)) + 1) << xl;
    for (int k = u0 + lane; k < u1; k += 64) {
      const int ul = 2 * wl - 4, img = k >> ul;
      const Unit u = unit_at((size_t)img * Cch + c, k & ((1 << ul) - 1), wl);
      const size_t o0 = u.plane + u.p, o1 = o0 + (1 << wl);
      const bf16x8_t a0 = ld8(r + o0), a1 = ld8(r + o1);
      float d[2][8];
      pool_relu_unit<POOLED, DENSE>(C, S, B, MN, c, img, gl, wl, u, a0, a1, d);
      const int at = (img << (2 * wl)) + u.p;   // the unit's first pixel in the channel
      if (at >= a && at < b) {                  // a unit's pixels may lie in two runs: one of them stores it
        bf16x8_t b0, b1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          b0[j] = to_bf16(d[0][j]);
          b1[j] = to_bf16(d[1][j]);
        }
        st8(dzb + o0, b0);
        st8(dzb + o1, b1);
      }
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int i = at + (y << wl) + j - a;
          if (i >= 0 && i < b - a) run[wv][i] = d[y][j];
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int j = 0; j < PRB_RUN / 64; ++j)
      if (64 * j + lane < b - a) acc[j & 3] += run[wv][64 * j + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  float s = (acc[0] + acc[2]) + (acc[1] + acc[3]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);   // lane i < o: entry i + entry i + o
  if (lane == 0) bpart[c * BP_PARTS + slice] = s;
}

// dense hidden-layer backward: dz[b][i] = C[i][b] * (h[b][i] > 0)
__global__ void k_relu_bwd_fc(const float* __restrict__ C, int S, int In, int B, const bf16* __restrict__ h,
                              float* __restrict__ dz, bf16* __restrict__ dzb) {
  const int total = In * B;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int f = i % In, b = i / In;
    const float g = from_bf16(h[i]) > 0.f ? split_sum(C, S, (size_t)In * B, (size_t)f * B + b) : 0.f;
    dz[i] = g;
    dzb[i] = to_bf16(g);
  }
}

// bias gradient: db[c] = sum over images and positions of dz[img][c][p] (one block per channel)
__global__ __launch_bounds__(256) void k_bias_grad(const float* __restrict__ dz, int B, int Cch, int HW,
                                                   float* __restrict__ db) {
  __shared__ float sh[256];
  const int c = blockIdx.x;
  float s = 0.f;
  for (int i = threadIdx.x; i < B * HW; i += 256) {
    const int img = i / HW, p = i - img * HW;
    s += dz[((size_t)img * Cch + c) * HW + p];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) db[c] = sh[0];
}

// MSE loss over the batch: dy = 2 (y - t) / (B*27); loss written by one block
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ y, const float* __restrict__ t, int n,
                                             float* __restrict__ dy, bf16* __restrict__ dyb,
                                             float* __restrict__ loss) {
  __shared__ float sh[256];
  float s = 0.f;
#pragma unroll 8
  for (int i = threadIdx.x; i < n; i += 256) {
    const float d = y[i] - t[i];
    s += d * d;
    const float g = 2.f * d / (float)n;
    dy[i] = g;
    dyb[i] = to_bf16(g);
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = sh[0] / (float)n;
}

__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, bf16* __restrict__ wb, int n, float lr, float b1, float b2,
                       float c1, float c2, float eps) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    wb[i] = to_bf16(wi);
  }
}

// The weights of the convolution layers 1 .. 3 as k_conv3's fragments, a layer per blockIdx.y (one launch for
// all, 4.6 us each): for the forward products (y < 3) A[m][k] = W[co = m][ci*9+kk], k = kk*Cin + ci,
// and for the data-gradient ones A[m][k] = W[co][ci = m][kk], k = kk*Cout + co; stored so that the 16 x 32
// fragment of K step s and row block b is one run of 512 values, 8 per lane, at (s * rows/16 + b) * 512.
struct ConvWeights {
  int off[3], cin[3], cout[3];
  int off1;   // of the first layer's fragments in wf
};
constexpr int C1_FRAG = 2 * (C1_OUT / 16) * 512;
__global__ void k_conv_weights(const bf16* __restrict__ wb, ConvWeights L, bf16* __restrict__ wf,
                               bf16* __restrict__ wt) {
  if (blockIdx.y == 0) {   // the first layer's: k = ci*9+kk, zeros from 45 to 63
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < C1_FRAG; i += gridDim.x * blockDim.x) {
      const int frag = i >> 9, lane = (i >> 3) & 63, m = (frag & 1) * 16 + (lane & 15);
      const int k = (frag >> 1) * 32 + (lane >> 4) * 8 + (i & 7);
      wf[L.off1 + i] = k < C1_K ? wb[m * C1_K + k] : (bf16)0.f;
    }
  }
  const int l = blockIdx.y % 3, Cin = L.cin[l], Cout = L.cout[l], n = Cin * Cout * 9;
  const bool fwd = blockIdx.y < 3;
  const int rows = fwd ? Cout : Cin, inner = fwd ? Cin : Cout;
  const bf16* W = wb + L.off[l];
  bf16* out = (fwd ? wf : wt) + L.off[l];
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int frag = i >> 9, lane = (i >> 3) & 63, step = frag / (rows >> 4), blk = frag - step * (rows >> 4);
    const int m = blk * 16 + (lane & 15), k = step * 32 + (lane >> 4) * 8 + (i & 7);
    const int kk = k / inner, c = k - kk * inner;
    const int co = fwd ? m : c, ci = fwd ? c : m;
    out[i] = W[((size_t)co * Cin + ci) * 9 + kk];
  }
}

__global__ void k_to_bf16(const float* __restrict__ w, bf16* __restrict__ wb, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) wb[i] = to_bf16(w[i]);
}

__global__ void k_acc_loss(const float* __restrict__ loss, float* __restrict__ acc) { *acc += *loss; }

// network output (standardised) -> unconstrained coordinates: psi = mean + std * y
__global__ void k_destandardise(const float* __restrict__ y, const float* __restrict__ mean,
                                const float* __restrict__ sd, int n, float* __restrict__ out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int j = i % 27;
    out[i] = mean[j] + sd[j] * y[i];
  }
}

// minibatch gather: xb[i] = x[order[i]], tb[i] = t[order[i]]
__global__ void k_gather(const bf16* __restrict__ x, const float* __restrict__ t, const int* __restrict__ order,
                         int B, int xsz, int tsz, bf16* __restrict__ xb, float* __restrict__ tb) {
  const int i = blockIdx.x;
  const size_t src = (size_t)order[i];
  for (int k = threadIdx.x; k < xsz; k += blockDim.x) xb[(size_t)i * xsz + k] = x[src * xsz + k];
  for (int k = threadIdx.x; k < tsz; k += blockDim.x) tb[(size_t)i * tsz + k] = t[src * tsz + k];
}

// Network input: for each source and band, the first image of that band, centre-cropped
// (or zero-padded) to 32x32 around the catalog position, scaled as (x - sky) / sqrt(sky).
__global__ __launch_bounds__(256) void k_patches(const SrcDev* __restrict__ srcs, const ImgDev* __restrict__ imgs,
                                                 const double* __restrict__ theta, bf16* __restrict__ out) {
  const int s = blockIdx.x;
  const double ux = theta[(size_t)s * NP], uy = theta[(size_t)s * NP + 1];
  for (int b = 0; b < 5; ++b) {
    int sel = -1;
    for (int i = srcs[s].img_begin; i < srcs[s].img_end; ++i)
      if (imgs[i].band == b) {
        sel = i;
        break;
      }
    bf16* o = out + ((size_t)s * 5 + b) * 1024;
    if (sel < 0) {
      for (int k = threadIdx.x; k < 1024; k += 256) o[k] = to_bf16(0.f);
      continue;
    }
    const ImgDev& im = imgs[sel];
    const double px = im.wcs[0] * ux + im.wcs[1] * uy + im.wcs[4] - im.origin[0];
    const double py = im.wcs[2] * ux + im.wcs[3] * uy + im.wcs[5] - im.origin[1];
    const int c0 = (int)floor(px + 0.5) - 16, r0 = (int)floor(py + 0.5) - 16;
    const float inv = (float)(1.0 / sqrt(im.sky));
    for (int k = threadIdx.x; k < 1024; k += 256) {
      const int r = r0 + k / 32, c = c0 + k % 32;
      float v = 0.f;
      if (r >= 0 && r < im.h && c >= 0 && c < im.w)
        v = ((float)im.pix[(size_t)r * im.pitch + c] - (float)im.sky) * inv;
      o[k] = to_bf16(v);
    }
  }
}

// Launches the product with at most `splits` K-splits; *splits is set to the number used
// (the count the epilogue must sum).
template <class LD>
hipError_t gemm(LD ld, int M, int N, int K, float* C, int& splits, hipStream_t st) {
  const int kchunk = ((K + splits - 1) / splits + TK - 1) / TK * TK;
  const int S = (K + kchunk - 1) / kchunk;
  splits = S;
  dim3 grid((N + TN - 1) / TN, (M + TM - 1) / TM, S);
  hipLaunchKernelGGL(k_gemm<LD>, grid, dim3(256), 0, st, ld, M, N, K, kchunk, C);
  return hipGetLastError();
}

// A weight gradient: the product's splits summed into gw (one split is written there directly), and, for a
// convolution (bpart), the bias gradient of its M channels from their slices.
template <class LD>
hipError_t gemm_sum(LD ld, int M, int N, int K, float* C, int splits, float* gw, hipStream_t st,
                    const float* bpart = nullptr, float* gb = nullptr) {
  const bool direct = splits == 1;
  const hipError_t e = gemm(ld, M, N, K, direct ? gw : C, splits, st);
  if (e != hipSuccess) return e;
  const int bw = direct ? 0 : (M * N + GS_COLS - 1) / GS_COLS, bb = bpart ? (M + 255) / 256 : 0;
  if (bw + bb > 0)
    hipLaunchKernelGGL(k_grad_sum, dim3(bw + bb), dim3(256), 0, st, C, splits, M * N, bw, gw, bpart, M, gb);
  return hipGetLastError();
}

inline int nblk(size_t n) { return (int)std::min<size_t>((n + 255) / 256, 16384); }

inline int ilog2(int v) {
  int l = 0;
  while ((1 << (l + 1)) <= v) ++l;
  return l;
}

// A k_conv3 product of M output channels over B images, its sums in `splits` K splits (the rule of gemm).
// Blocks of 256 pixels where that leaves two blocks or more per compute unit, else (and where
// the sums of splits must be kept beside the running ones, or 128 channels would take 109 KB of LDS)
// of 128.
template <int CL, int WL, int MF, bool FLIP>
hipError_t conv3(const bf16* wfrag, const bf16* X, int B, int M, int splits, const float* bias, bf16* act, bf16* pool,
                 float* out, hipStream_t st) {
  constexpr int K = 9 << CL;
  const int chunk = ((K + splits - 1) / splits + TK - 1) / TK;
  const int64_t n = (int64_t)B << (2 * WL);
  const int rows = M / (16 * MF);
  if (M != rows * 16 * MF) return hipErrorInvalidValue;
  if constexpr (CL < 7)
    if (splits == 1 && (n + 255) / 256 * rows >= 512) {
      hipLaunchKernelGGL((k_conv3<CL, WL, MF, 4, FLIP>), dim3((n + 255) / 256, rows), dim3(256), 0, st, wfrag, X, B, M,
                         chunk, bias, act, pool, out);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((k_conv3<CL, WL, MF, 2, FLIP>), dim3((n + 127) / 128, rows), dim3(256), 0, st, wfrag, X, B, M, chunk,
                     bias, act, pool, out);
  return hipGetLastError();
}

}  // namespace

// ============================================================ network object (host side)

struct NetLayout {
  static constexpr int NCONV = 4;
  int cin[4] = {5, 32, 64, 64}, cout[4] = {32, 64, 64, 128}, hw[4] = {32, 32, 16, 8};
  int pool[4] = {0, 1, 1, 1};
  size_t off[12];
  size_t total = 0;
  NetLayout() {
    size_t o = 0;
    for (int l = 0; l < 4; ++l) {
      off[2 * l] = o;
      o += (size_t)cout[l] * cin[l] * 9;
      off[2 * l + 1] = o;
      o += cout[l];
    }
    off[8] = o;
    o += 256 * 2048;
    off[9] = o;
    o += 256;
    off[10] = o;
    o += 27 * 256;
    off[11] = o;
    o += 27;
    total = o;
  }
};

struct NetState {
  NetLayout L;
  float* w = nullptr;     // FP32 master weights
  float* m = nullptr;     // Adam moments
  float* v = nullptr;
  float* g = nullptr;     // gradient
  bf16* wb = nullptr;     // BF16 weights
  bf16* wt = nullptr;     // convolution weights re-laid for the data-gradient products (conv offsets)
  bf16* wf = nullptr;     // ... for the forward products (conv offsets; the first layer's after the others)
  int step = 0;
  int cap_batch = 0;
  // activations (BF16) and gradients for cap_batch images
  bf16 *x = nullptr, *r[4] = {}, *p[4] = {}, *h = nullptr, *dyb = nullptr, *dzb = nullptr, *dhb = nullptr;
  float *y = nullptr, *t = nullptr, *dy = nullptr, *dh = nullptr, *C = nullptr, *loss = nullptr;
  float* bpart = nullptr;   // conv bias-gradient slices (128 channels x BP_PARTS)
  size_t c_cap = 0;
};

hipError_t net_alloc(NetState* n) {
  const size_t P = n->L.total;
  hipError_t e;
  if ((e = hipMalloc(&n->w, P * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->m, P * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->v, P * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->g, P * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->wb, P * 2)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->wt, n->L.off[8] * 2)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->wf, (n->L.off[8] + C1_FRAG) * 2)) != hipSuccess) return e;
  if ((e = hipMemset(n->m, 0, P * 4)) != hipSuccess) return e;
  if ((e = hipMemset(n->v, 0, P * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&n->bpart, sizeof(float) * 128 * BP_PARTS)) != hipSuccess) return e;
  return hipMalloc(&n->loss, 16);
}

void net_free_work(NetState* n) {
  bf16* bb[] = {n->x, n->r[0], n->r[1], n->r[2], n->r[3], n->p[0], n->p[1], n->p[2], n->p[3], n->h, n->dyb,
                n->dzb, n->dhb};
  for (bf16* q : bb)
    if (q) (void)hipFree(q);
  float* ff[] = {n->y, n->t, n->dy, n->dh, n->C};
  for (float* q : ff)
    if (q) (void)hipFree(q);
  n->x = n->h = n->dyb = n->dzb = n->dhb = nullptr;
  for (int l = 0; l < 4; ++l) n->r[l] = n->p[l] = nullptr;
  n->y = n->t = n->dy = n->dh = n->C = nullptr;
  n->cap_batch = 0;
}

void net_free(NetState* n) {
  net_free_work(n);
  float* ff[] = {n->w, n->m, n->v, n->g, n->loss, n->bpart};
  for (float* q : ff)
    if (q) (void)hipFree(q);
  if (n->wb) (void)hipFree(n->wb);
  if (n->wt) (void)hipFree(n->wt);
  if (n->wf) (void)hipFree(n->wf);
}

static const int kSplitTarget = 1024;   // aim for about this many GEMM blocks

hipError_t net_reserve(NetState* n, int B) {
  if (B <= n->cap_batch) return hipSuccess;
  net_free_work(n);
  const NetLayout& L = n->L;
  hipError_t e;
#define ALLOC(ptr, bytes) \
  if ((e = hipMalloc(&(ptr), (bytes))) != hipSuccess) return e
  ALLOC(n->x, (size_t)B * 5 * 1024 * 2);
  size_t maxact = 0;
  for (int l = 0; l < 4; ++l) {
    const size_t a = (size_t)B * L.cout[l] * L.hw[l] * L.hw[l];
    ALLOC(n->r[l], a * 2);
    const int ho = L.pool[l] ? L.hw[l] / 2 : L.hw[l];
    ALLOC(n->p[l], (size_t)B * L.cout[l] * ho * ho * 2);
    maxact = std::max(maxact, a);
  }
  ALLOC(n->h, (size_t)B * 256 * 2);
  ALLOC(n->dyb, (size_t)B * 27 * 2);
  ALLOC(n->dzb, maxact * 2);
  ALLOC(n->dhb, (size_t)B * 256 * 2);
  ALLOC(n->y, (size_t)B * 27 * 4);
  ALLOC(n->t, (size_t)B * 27 * 4);
  ALLOC(n->dy, (size_t)B * 27 * 4);
  ALLOC(n->dh, (size_t)B * 2048 * 4);
  // split-K partial products: the largest M*N times the split count
  n->c_cap = std::max(maxact * 2, (size_t)8 << 20);
  ALLOC(n->C, n->c_cap * 4);
#undef ALLOC
  n->cap_batch = B;
  return hipSuccess;
}

static int splits_for(size_t M, size_t N, size_t K, size_t cap, size_t tn = 64) {
  const size_t blocks = ((M + TM - 1) / TM) * ((N + tn - 1) / tn);
  int s = 1;
  while (blocks * s < (size_t)kSplitTarget && K / (size_t)(s * 2) >= 256 && (size_t)(s * 2) * M * N <= cap) s *= 2;
  return s;
}

// Forward pass of B images at x_in (BF16, B x 5 x 32 x 32); leaves y (FP32, B x 27), and the weights that
// net_backward reads in n->wt where it follows (backward).
hipError_t net_forward(NetState* n, const bf16* x_in, int B, hipStream_t st, bool backward) {
  const NetLayout& L = n->L;
  hipError_t e;
  ConvWeights cw;
  cw.off1 = (int)L.off[8];
  for (int l = 1; l < 4; ++l) {
    cw.off[l - 1] = (int)L.off[2 * l];
    cw.cin[l - 1] = L.cin[l];
    cw.cout[l - 1] = L.cout[l];
  }
  hipLaunchKernelGGL(k_conv_weights, dim3(nblk((size_t)128 * 64 * 9), backward ? 6 : 3), dim3(256), 0, st, n->wb, cw,
                     n->wf, n->wt);
  const auto splits = [&](int l) {
    return splits_for(L.cout[l], (size_t)B * L.hw[l] * L.hw[l], (size_t)L.cin[l] * 9, n->c_cap, 128);
  };
  const auto act = [&](int l) { return backward || !L.pool[l] ? n->r[l] : nullptr; };   // the backward pass reads it
  const auto bias = [&](int l) { return n->w + L.off[2 * l + 1]; };
  hipLaunchKernelGGL(k_conv1, dim3(4 * B), dim3(256), 0, st, n->wf + cw.off1, x_in, bias(0), n->r[0]);
  if ((e = conv3<5, 5, 4, false>(n->wf + L.off[2], n->r[0], B, 64, splits(1), bias(1), act(1), n->p[1], nullptr, st)) !=
      hipSuccess)
    return e;
  if ((e = conv3<6, 4, 4, false>(n->wf + L.off[4], n->p[1], B, 64, splits(2), bias(2), act(2), n->p[2], nullptr, st)) !=
      hipSuccess)
    return e;
  if ((e = conv3<6, 3, 4, false>(n->wf + L.off[6], n->p[2], B, 128, splits(3), bias(3), act(3), n->p[3], nullptr, st)) !=
      hipSuccess)
    return e;
  const bf16* in = n->p[3];
  {
    int S = splits_for(256, B, 2048, n->c_cap);
    LdFcFwd ld{n->wb + L.off[8], in, 2048};
    if ((e = gemm(ld, 256, B, 2048, n->C, S, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_ep_fc_fwd, dim3(nblk((size_t)256 * B)), dim3(256), 0, st, n->C, S, 256, B,
                       n->w + L.off[9], n->h, (float*)nullptr);
  }
  {
    int S = splits_for(27, B, 256, n->c_cap);
    LdFcFwd ld{n->wb + L.off[10], n->h, 256};
    if ((e = gemm(ld, 27, B, 256, n->C, S, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_ep_fc_fwd, dim3(nblk((size_t)27 * B)), dim3(256), 0, st, n->C, S, 27, B,
                       n->w + L.off[11], (bf16*)nullptr, n->y);
  }
  return hipGetLastError();
}

// Loss and full gradient (into n->g) for the B images at x_in (the forward input) with
// targets in n->t.
hipError_t net_backward(NetState* n, const bf16* x_in, int B, hipStream_t st) {
  const NetLayout& L = n->L;
  hipError_t e;
  hipLaunchKernelGGL(k_mse, dim3(1), dim3(256), 0, st, n->y, n->t, B * 27, n->dy, n->dyb, n->loss);
  // dense output layer
  {
    int S = splits_for(27, 256, B, n->c_cap);
    LdFcWgrad ld{n->dyb, n->h, 256, 27};
    if ((e = gemm_sum(ld, 27, 256, B, n->C, S, n->g + L.off[10], st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_bias_grad, dim3(27), dim3(256), 0, st, n->dy, B, 27, 1, n->g + L.off[11]);
    int S2 = splits_for(256, B, 27, n->c_cap);
    LdFcDgrad ld2{n->wb + L.off[10], n->dyb, 256, 27};
    if ((e = gemm(ld2, 256, B, 27, n->C, S2, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_relu_bwd_fc, dim3(nblk((size_t)256 * B)), dim3(256), 0, st, n->C, S2, 256, B, n->h, n->dh,
                       n->dhb);
  }
  // dense hidden layer
  {
    int S = splits_for(256, 2048, B, n->c_cap);
    LdFcWgrad ld{n->dhb, n->p[3], 2048, 256};
    if ((e = gemm_sum(ld, 256, 2048, B, n->C, S, n->g + L.off[8], st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_bias_grad, dim3(256), dim3(256), 0, st, n->dh, B, 256, 1, n->g + L.off[9]);
    int S2 = splits_for(2048, B, 256, n->c_cap);
    LdFcDgrad ld2{n->wb + L.off[8], n->dhb, 2048, 256};
    if ((e = gemm(ld2, 2048, B, 256, n->C, S2, st)) != hipSuccess) return e;
    // into conv4's post-ReLU activation through its pool (dense layout C[c*16+q][img])
    hipLaunchKernelGGL((k_pool_relu_bwd<true, true>), dim3(BP_PARTS / 4, 128), dim3(256), 0, st, n->C, S2, B, 128,
                       3, n->r[3], n->dzb, n->bpart);
  }
  for (int l = 3; l >= 0; --l) {
    const int HW = L.hw[l] * L.hw[l];
    const bf16* xin = l == 0 ? x_in : (L.pool[l - 1] ? n->p[l - 1] : n->r[l - 1]);
    // weight and bias gradients
    {
      const size_t M = L.cout[l], N = (size_t)L.cin[l] * 9, K = (size_t)B * HW;
      int S = splits_for(M, N, K, n->c_cap);
      const int wl = ilog2(L.hw[l]);
      LdConvWgrad ld{n->dzb, xin, L.cin[l], L.cout[l], 2 * wl, wl};
      if ((e = gemm_sum(ld, (int)M, (int)N, (int)K, n->C, S, n->g + L.off[2 * l], st, n->bpart,
                        n->g + L.off[2 * l + 1])) != hipSuccess)
        return e;
    }
    if (l == 0) break;
    // data gradient into the previous layer's post-ReLU activation (through its pool)
    {
      const int M = L.cin[l];
      const int S = splits_for(M, (size_t)B * HW, (size_t)L.cout[l] * 9, n->c_cap, 128);
      const bf16* wt = n->wt + L.off[2 * l];
      e = l == 3   ? conv3<7, 3, 4, true>(wt, n->dzb, B, M, S, nullptr, nullptr, nullptr, n->C, st)
          : l == 2 ? conv3<6, 4, 4, true>(wt, n->dzb, B, M, S, nullptr, nullptr, nullptr, n->C, st)
                   : conv3<6, 5, 2, true>(wt, n->dzb, B, M, S, nullptr, nullptr, nullptr, n->C, st);
      if (e != hipSuccess) return e;
      const int wlp = ilog2(L.hw[l - 1]);
      const auto k = L.pool[l - 1] ? &k_pool_relu_bwd<true, false> : &k_pool_relu_bwd<false, false>;
      hipLaunchKernelGGL(k, dim3(BP_PARTS / 4, L.cout[l - 1]), dim3(256), 0, st, n->C, 1, B, L.cout[l - 1], wlp,
                         n->r[l - 1], n->dzb, n->bpart);
    }
  }
  return hipGetLastError();
}

hipError_t net_adam(NetState* n, float lr, hipStream_t st) {
  n->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - powf(b1, (float)n->step), c2 = 1.f - powf(b2, (float)n->step);
  hipLaunchKernelGGL(k_adam, dim3(nblk(n->L.total)), dim3(256), 0, st, n->w, n->m, n->v, n->g, n->wb,
                     (int)n->L.total, lr, b1, b2, c1, c2, 1e-8f);
  return hipGetLastError();
}

hipError_t net_sync_bf16(NetState* n, hipStream_t st) {
  hipLaunchKernelGGL(k_to_bf16, dim3(nblk(n->L.total)), dim3(256), 0, st, n->w, n->wb, (int)n->L.total);
  return hipGetLastError();
}

hipError_t net_gather(NetState* n, const void* x, const float* t, const int* order, int B, hipStream_t st) {
  hipLaunchKernelGGL(k_gather, dim3(B), dim3(256), 0, st, (const bf16*)x, t, order, B, 5 * 1024, t ? 27 : 0, n->x,
                     n->t);
  return hipGetLastError();
}

hipError_t net_acc_loss(NetState* n, float* acc, hipStream_t st) {
  hipLaunchKernelGGL(k_acc_loss, dim3(1), dim3(1), 0, st, n->loss, acc);
  return hipGetLastError();
}

hipError_t launch_patches(const SrcDev* srcs, int n_src, const ImgDev* imgs, const double* theta, void* out,
                          hipStream_t st) {
  if (n_src <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_patches, dim3(n_src), dim3(256), 0, st, srcs, imgs, theta, (bf16*)out);
  return hipGetLastError();
}

hipError_t net_destandardise(const float* y, const float* mean, const float* sd, int n, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_destandardise, dim3(nblk(n)), dim3(256), 0, st, y, mean, sd, n, out);
  return hipGetLastError();
}

}  // namespace celeste

// ============================================================ C ABI of the network

using celeste::NetState;

struct celeste_net {
  NetState s;
  int device = 0;
  hipStream_t stream = nullptr;
  float* psi_mean = nullptr;   // device, 27
  float* psi_std = nullptr;    // device, 27
  float* acc = nullptr;        // device per-epoch loss accumulators
  int acc_cap = 0;
  void* patches = nullptr;     // device BF16 inputs for inference inside fits
  size_t patches_cap = 0;
};

namespace {
thread_local std::string g_net_err;
int net_fail(int code, const char* msg, hipError_t e = hipSuccess) {
  g_net_err = msg;
  if (e != hipSuccess) {
    g_net_err += ": ";
    g_net_err += hipGetErrorString(e);
  }
  celeste::set_error(g_net_err.c_str());
  return code;
}
#define NETCHK(x, msg)                                     \
  do {                                                     \
    hipError_t e_ = (x);                                   \
    if (e_ != hipSuccess) return net_fail(CELESTE_E_DEVICE, msg, e_); \
  } while (0)
}  // namespace

namespace celeste {

// Predicted start for each source of a packed batch: patches around the catalog
// positions (theta's u), network forward in chunks, and psi = mean + std * y.
int surrogate_predict(celeste_net* net, const SrcDev* srcs, int n_src, const ImgDev* imgs, const double* theta_cat,
                      float* psi_out, hipStream_t st) {
  const size_t need = (size_t)n_src * 5 * 1024 * 2;
  if (need > net->patches_cap) {
    if (net->patches) (void)hipFree(net->patches);
    net->patches = nullptr;
    net->patches_cap = 0;
    NETCHK(hipMalloc(&net->patches, need), "surrogate patch buffer");
    net->patches_cap = need;
  }
  NETCHK(launch_patches(srcs, n_src, imgs, theta_cat, net->patches, st), "patch extraction");
  const int chunk = 4096;
  NETCHK(net_reserve(&net->s, std::min(chunk, n_src)), "network workspace");
  for (int a = 0; a < n_src; a += chunk) {
    const int B = std::min(chunk, n_src - a);
    NETCHK(net_forward(&net->s, (const bf16*)net->patches + (size_t)a * 5 * 1024, B, st, false), "network forward");
    NETCHK(net_destandardise(net->s.y, net->psi_mean, net->psi_std, B * 27, psi_out + (size_t)a * 27, st),
           "destandardise");
  }
  return CELESTE_OK;
}

}  // namespace celeste

extern "C" {

int64_t celeste_net_num_params(void) { return (int64_t)celeste::NetLayout().total; }

int celeste_net_create(celeste_ctx* ctx, const float* params, int64_t n_params, const float* psi_mean,
                       const float* psi_std, celeste_net** out) {
  if (!ctx || !params || !psi_mean || !psi_std || !out) return net_fail(CELESTE_E_INVALID, "NULL argument");
  *out = nullptr;
  celeste_net* net = new (std::nothrow) celeste_net();
  if (!net) return net_fail(CELESTE_E_NOMEM, "network allocation");
  if (n_params != (int64_t)net->s.L.total) {
    delete net;
    return net_fail(CELESTE_E_INVALID, "parameter count does not match the network");
  }
  for (int j = 0; j < 27; ++j)
    if (!(psi_std[j] > 0.f) || !std::isfinite(psi_mean[j])) {
      delete net;
      return net_fail(CELESTE_E_INVALID, "psi_std must be positive and psi_mean finite");
    }
  net->device = celeste::ctx_device(ctx);
  net->stream = celeste::ctx_stream(ctx);
  hipError_t e = hipSetDevice(net->device);
  if (e == hipSuccess) e = celeste::net_alloc(&net->s);
  if (e == hipSuccess) e = hipMalloc(&net->psi_mean, 27 * 4);
  if (e == hipSuccess) e = hipMalloc(&net->psi_std, 27 * 4);
  if (e == hipSuccess) e = hipMemcpy(net->s.w, params, net->s.L.total * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(net->psi_mean, psi_mean, 27 * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(net->psi_std, psi_std, 27 * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = celeste::net_sync_bf16(&net->s, net->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(net->stream);
  if (e != hipSuccess) {
    celeste::net_free(&net->s);
    delete net;
    return net_fail(CELESTE_E_DEVICE, "network set-up", e);
  }
  *out = net;
  return CELESTE_OK;
}

void celeste_net_destroy(celeste_net* net) {
  if (!net) return;
  (void)hipSetDevice(net->device);
  (void)hipStreamSynchronize(net->stream);
  celeste::net_free(&net->s);
  if (net->psi_mean) (void)hipFree(net->psi_mean);
  if (net->psi_std) (void)hipFree(net->psi_std);
  if (net->acc) (void)hipFree(net->acc);
  if (net->patches) (void)hipFree(net->patches);
  delete net;
}

int celeste_net_get_params(celeste_net* net, float* out) {
  if (!net || !out) return net_fail(CELESTE_E_INVALID, "NULL argument");
  NETCHK(hipSetDevice(net->device), "set device");
  NETCHK(hipStreamSynchronize(net->stream), "sync");
  NETCHK(hipMemcpy(out, net->s.w, net->s.L.total * 4, hipMemcpyDeviceToHost), "read parameters");
  return CELESTE_OK;
}

int celeste_net_loss_grad(celeste_net* net, const void* x, const float* t, int batch, float* loss, float* grad) {
  if (!net || !x || !t || !loss || batch < 1) return net_fail(CELESTE_E_INVALID, "bad argument");
  if ((reinterpret_cast<uintptr_t>(x) & 15) != 0) return net_fail(CELESTE_E_INVALID, "x must be 16-byte aligned");
  NETCHK(hipSetDevice(net->device), "set device");
  hipStream_t st = net->stream;
  NETCHK(celeste::net_reserve(&net->s, batch), "network workspace");
  NETCHK(hipMemcpyAsync(net->s.t, t, (size_t)batch * 27 * 4, hipMemcpyDeviceToDevice, st), "targets");
  NETCHK(celeste::net_forward(&net->s, (const celeste::bf16*)x, batch, st, true), "forward");
  NETCHK(celeste::net_backward(&net->s, (const celeste::bf16*)x, batch, st), "backward");
  NETCHK(hipMemcpyAsync(loss, net->s.loss, 4, hipMemcpyDeviceToHost, st), "loss");
  if (grad) NETCHK(hipMemcpyAsync(grad, net->s.g, net->s.L.total * 4, hipMemcpyDeviceToHost, st), "gradient");
  NETCHK(hipStreamSynchronize(st), "sync");
  return CELESTE_OK;
}

int celeste_net_forward(celeste_net* net, const void* x, int64_t n, float* y) {
  if (!net || !x || !y || n < 1) return net_fail(CELESTE_E_INVALID, "bad argument");
  if ((reinterpret_cast<uintptr_t>(x) & 15) != 0) return net_fail(CELESTE_E_INVALID, "x must be 16-byte aligned");
  NETCHK(hipSetDevice(net->device), "set device");
  hipStream_t st = net->stream;
  const int chunk = 4096;
  NETCHK(celeste::net_reserve(&net->s, (int)std::min<int64_t>(chunk, n)), "network workspace");
  for (int64_t a = 0; a < n; a += chunk) {
    const int B = (int)std::min<int64_t>(chunk, n - a);
    NETCHK(celeste::net_forward(&net->s, (const celeste::bf16*)x + a * 5 * 1024, B, st, false), "forward");
    NETCHK(hipMemcpyAsync(y + a * 27, net->s.y, (size_t)B * 27 * 4, hipMemcpyDeviceToDevice, st), "output");
  }
  NETCHK(hipStreamSynchronize(st), "sync");
  return CELESTE_OK;
}

int celeste_net_train(celeste_net* net, const void* x, const float* t, int64_t n, const int32_t* orders, int epochs,
                      int batch, float lr, float* epoch_loss) {
  if (!net || !x || !t || !orders || n < 1 || epochs < 1 || batch < 1 || !(lr > 0.f))
    return net_fail(CELESTE_E_INVALID, "bad argument");
  NETCHK(hipSetDevice(net->device), "set device");
  hipStream_t st = net->stream;
  NETCHK(celeste::net_reserve(&net->s, batch), "network workspace");
  if (epochs > net->acc_cap) {
    if (net->acc) (void)hipFree(net->acc);
    net->acc = nullptr;
    NETCHK(hipMalloc(&net->acc, (size_t)epochs * 4), "loss accumulators");
    net->acc_cap = epochs;
  }
  NETCHK(hipMemsetAsync(net->acc, 0, (size_t)epochs * 4, st), "zero accumulators");
  const int64_t nb = (n + batch - 1) / batch;
  for (int e = 0; e < epochs; ++e) {
    for (int64_t b = 0; b < nb; ++b) {
      const int B = (int)std::min<int64_t>(batch, n - b * batch);
      NETCHK(celeste::net_gather(&net->s, x, t, (const int*)orders + (size_t)e * n + b * batch, B, st), "gather");
      NETCHK(celeste::net_forward(&net->s, net->s.x, B, st, true), "forward");
      NETCHK(celeste::net_backward(&net->s, net->s.x, B, st), "backward");
      NETCHK(celeste::net_adam(&net->s, lr, st), "adam");
      NETCHK(celeste::net_acc_loss(&net->s, net->acc + e, st), "loss");
    }
  }
  if (epoch_loss) {
    NETCHK(hipMemcpyAsync(epoch_loss, net->acc, (size_t)epochs * 4, hipMemcpyDeviceToHost, st), "losses");
    NETCHK(hipStreamSynchronize(st), "sync");
    for (int e = 0; e < epochs; ++e) epoch_loss[e] /= (float)nb;
  }
  NETCHK(hipStreamSynchronize(st), "sync");
  return CELESTE_OK;
}

}  // extern "C"
