// Per-image setup, per-image constants, pixel validation and the plain start.
//
// The setup kernel turns one source's parameters into the FP32 table its pixel
// work reads (section III-A model; III-B objective): the source position in the
// patch, the brightness moments of the Bernoulli/lognormal mixture in the image's
// band, the covariance precision and normaliser of every star and galaxy mixture
// component after convolution with the image's PSF, and the coefficients that map
// position-space Hermite moments onto derivatives with respect to the galaxy shape.
// All of this is computed in FP64 and rounded once to FP32.
#include <math.h>

#include "celeste_internal.h"
#include "tiles.h"

namespace celeste {

namespace {

// log l_b = log l_r + S_b . c, colours c_j = log(l_{j+1} / l_j), bands u,g,r,i,z.
__device__ __constant__ double kColourSigns[5][4] = {
    {-1.0, -1.0, 0.0, 0.0}, {0.0, -1.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 1.0, 0.0}, {0.0, 0.0, 1.0, 1.0}};

constexpr double kLog2e = 1.4426950408889634;
constexpr double kTwoPi = 6.283185307179586;

struct Sym2 {
  double xx, xy, yy;
};

// A X A^T for symmetric X.
__device__ inline Sym2 congruence(const double* wcs, Sym2 X) {
  const double a00 = wcs[0], a01 = wcs[1], a10 = wcs[2], a11 = wcs[3];
  // rows of A X
  const double r0x = a00 * X.xx + a01 * X.xy, r0y = a00 * X.xy + a01 * X.yy;
  const double r1x = a10 * X.xx + a11 * X.xy, r1y = a10 * X.xy + a11 * X.yy;
  Sym2 o;
  o.xx = r0x * a00 + r0y * a01;
  o.xy = r0x * a10 + r0y * a11;
  o.yy = r1x * a10 + r1y * a11;
  return o;
}

struct ShapeDerivs {
  Sym2 W;         // shape matrix (image frame)
  Sym2 d[3];      // d/d(e_axis, e_angle, e_scale)
  Sym2 dd[6];     // pairs (0,0),(0,1),(0,2),(1,1),(1,2),(2,2)
};

// W = s^2 M(q,t), M = R(t) diag(1,q^2) R(t)^T, entries in closed form.
__device__ ShapeDerivs shape_derivs(double q, double t, double s, const double* wcs) {
  const double c = cos(t), sn = sin(t);
  const double c2t = cos(2.0 * t), s2t = sin(2.0 * t);
  const double omq = 1.0 - q * q;
  Sym2 M = {c * c + q * q * sn * sn, omq * c * sn, sn * sn + q * q * c * c};
  Sym2 Mq = {2.0 * q * sn * sn, -2.0 * q * c * sn, 2.0 * q * c * c};
  Sym2 Mt = {-omq * s2t, omq * c2t, omq * s2t};
  Sym2 Mqq = {2.0 * sn * sn, -2.0 * c * sn, 2.0 * c * c};
  Sym2 Mqt = {2.0 * q * s2t, -2.0 * q * c2t, -2.0 * q * s2t};
  Sym2 Mtt = {-2.0 * omq * c2t, -2.0 * omq * s2t, 2.0 * omq * c2t};
  auto sc = [](Sym2 a, double f) { return Sym2{a.xx * f, a.xy * f, a.yy * f}; };
  const double s2 = s * s;
  ShapeDerivs o;
  o.W = congruence(wcs, sc(M, s2));
  o.d[0] = congruence(wcs, sc(Mq, s2));
  o.d[1] = congruence(wcs, sc(Mt, s2));
  o.d[2] = congruence(wcs, sc(M, 2.0 * s));
  o.dd[0] = congruence(wcs, sc(Mqq, s2));
  o.dd[1] = congruence(wcs, sc(Mqt, s2));
  o.dd[2] = congruence(wcs, sc(Mq, 2.0 * s));
  o.dd[3] = congruence(wcs, sc(Mtt, s2));
  o.dd[4] = congruence(wcs, sc(Mt, 2.0 * s));
  o.dd[5] = congruence(wcs, sc(M, 2.0));
  return o;
}

// The exponent's constants of w N(0, C) and its precision.
__device__ inline Sym2 write_exponent(float* rec, double w, Sym2 C) {
  const double det = C.xx * C.yy - C.xy * C.xy;
  const double inv = 1.0 / det;
  const Sym2 P = {C.yy * inv, -C.xy * inv, C.xx * inv};
  rec[tab::R_C0] = (float)(log2(w) - log2(kTwoPi) - 0.5 * log2(det));
  rec[tab::R_QXX] = (float)(-0.5 * kLog2e * P.xx);
  rec[tab::R_QXY] = (float)(-kLog2e * P.xy);
  rec[tab::R_QYY] = (float)(-0.5 * kLog2e * P.yy);
  return P;
}

__device__ inline Sym2 write_gaussian(float* rec, double w, Sym2 C) {
  const Sym2 P = write_exponent(rec, w, C);
  rec[tab::R_PXX] = (float)P.xx;
  rec[tab::R_PXY] = (float)P.xy;
  rec[tab::R_PYY] = (float)P.yy;
  return P;
}

__device__ inline void write_galaxy(float* expo, float* rec, double w, Sym2 C, double nu) {
  const Sym2 P = write_gaussian(rec, w, C);
  for (int i = 0; i < tab::EXPO_REC; ++i) expo[i] = rec[i];
  rec[tab::R_NU] = (float)nu;
  rec[tab::R_3PXX] = (float)(3.0 * P.xx);
  rec[tab::R_3PYY] = (float)(3.0 * P.yy);
  rec[tab::R_2PXY] = (float)(2.0 * P.xy);
  rec[tab::R_6PXX] = (float)(6.0 * P.xx);
  rec[tab::R_6PYY] = (float)(6.0 * P.yy);
  rec[tab::R_3PXY] = (float)(3.0 * P.xy);
  rec[tab::R_4PXY] = (float)(4.0 * P.xy);
  rec[tab::R_K4A] = (float)(3.0 * P.xx * P.xx);
  rec[tab::R_K4B] = (float)(3.0 * P.xx * P.xy);
  rec[tab::R_K4C] = (float)(2.0 * P.xy * P.xy);
  rec[tab::R_K4D] = (float)(3.0 * P.yy * P.xy);
  rec[tab::R_K4E] = (float)(3.0 * P.yy * P.yy);
}

// One 64-thread block per image: thread 0 writes the header and the shape
// coefficients, thread k < n_psf a star component, the rest galaxy components.  Without DERIVS only
// what values and field rates read: no shape derivatives and no component records, a fifth of the table's bytes
// (60,000 images: 93 us, 151 us with all of it).
template <bool DERIVS>
__global__ __launch_bounds__(64) void k_setup(const ImgDev* __restrict__ imgs, const double* __restrict__ theta,
                                               const int* __restrict__ src_flag, ProfDev prof,
                                               float* __restrict__ tables, int tstride) {
  const int i = blockIdx.x;
  const ImgDev& im = imgs[i];
  const int s = im.src;
  if (src_flag && !src_flag[s]) return;
  const double* th = theta + (size_t)s * NP;
  float* T = tables + (size_t)i * tstride;
  const int t = threadIdx.x;
  const double e_dev = th[3], e_axis = th[4], e_angle = th[5], e_scale = th[6];
  const ShapeDerivs sd = shape_derivs(e_axis, e_angle, e_scale, im.wcs);
  const int ncomp = prof.n_exp + prof.n_dev;

  if (t == 0) {
    const double* S = kColourSigns[im.band];
    double m_s = th[7], v_s = th[9], m_g = th[8], v_g = th[10];
    for (int j = 0; j < 4; ++j) {
      m_s += S[j] * th[11 + j];
      v_s += S[j] * S[j] * th[19 + j];
      m_g += S[j] * th[15 + j];
      v_g += S[j] * S[j] * th[23 + j];
    }
    const double a = th[2];
    const double px = im.wcs[0] * th[0] + im.wcs[1] * th[1] + im.wcs[4];
    const double py = im.wcs[2] * th[0] + im.wcs[3] * th[1] + im.wcs[5];
    const double mu_s = exp(m_s + 0.5 * v_s), mu_g = exp(m_g + 0.5 * v_g);
    const double B_s = mu_s * mu_s, B_g = mu_g * mu_g;      // E[l]^2
    const double em_s = expm1(v_s), em_g = expm1(v_g);       // e^v - 1
    const double Ks = a * B_s * (em_s + (1.0 - a));
    const double Kg = (1.0 - a) * B_g * (em_g + a);
    const double Ksg = -2.0 * a * (1.0 - a) * mu_s * mu_g;
    const double Ka_s = B_s * (em_s + 1.0 - 2.0 * a);
    const double Ka_g = -B_g * (em_g + 2.0 * a - 1.0);
    const double Ka_sg = -2.0 * (1.0 - 2.0 * a) * mu_s * mu_g;
    const double Kv_s = a * B_s * (2.0 * em_s + 2.0 - a);
    const double Kv_g = (1.0 - a) * B_g * (2.0 * em_g + 1.0 + a);
    T[tab::PSX] = (float)(px - im.origin[0]);
    T[tab::PSY] = (float)(py - im.origin[1]);
    T[tab::CALIB] = (float)im.calib;
    T[tab::SKY] = (float)im.sky;
    T[tab::CS] = (float)(a * mu_s);
    T[tab::CG] = (float)((1.0 - a) * mu_g);
    T[tab::MU_S] = (float)mu_s;
    T[tab::MU_G] = (float)mu_g;
    T[tab::KS] = (float)Ks;
    T[tab::KG] = (float)Kg;
    T[tab::KSG] = (float)Ksg;
    T[tab::KA_S] = (float)Ka_s;
    T[tab::KA_G] = (float)Ka_g;
    T[tab::KA_SG] = (float)Ka_sg;
    T[tab::KV_S] = (float)Kv_s;
    T[tab::KV_G] = (float)Kv_g;
    T[tab::EDEV] = (float)e_dev;
    T[tab::KS_AA] = (float)(-2.0 * B_s);
    T[tab::KS_AM] = (float)(2.0 * Ka_s);
    T[tab::KS_AV] = (float)(2.0 * B_s * (em_s + 1.0 - a));
    T[tab::KS_MM] = (float)(4.0 * Ks);
    T[tab::KS_MV] = (float)(2.0 * Kv_s);
    T[tab::KS_VV] = (float)(a * B_s * (4.0 * em_s + 4.0 - a));
    T[tab::KG_AA] = (float)(-2.0 * B_g);
    T[tab::KG_AM] = (float)(2.0 * Ka_g);
    T[tab::KG_AV] = (float)(-2.0 * B_g * (em_g + a));
    T[tab::KG_MM] = (float)(4.0 * Kg);
    T[tab::KG_MV] = (float)(2.0 * Kv_g);
    T[tab::KG_VV] = (float)((1.0 - a) * B_g * (4.0 * em_g + 3.0 + a));
    T[tab::KSG_AA] = (float)(4.0 * mu_s * mu_g);
    T[tab::KSG_AM] = (float)Ka_sg;
    T[tab::KSG_AV] = (float)(0.5 * Ka_sg);
    T[tab::NPSF] = (float)im.n_psf;
    // shape contractions
    for (int e = 0; DERIVS && e < 3; ++e) {
      T[tab::W1 + 3 * e + 0] = (float)(0.5 * sd.d[e].xx);
      T[tab::W1 + 3 * e + 1] = (float)(sd.d[e].xy);
      T[tab::W1 + 3 * e + 2] = (float)(0.5 * sd.d[e].yy);
    }
    const int pa[6] = {0, 0, 0, 1, 1, 2}, pb[6] = {0, 1, 2, 1, 2, 2};
    for (int k = 0; DERIVS && k < 6; ++k) {
      const Sym2 U = sd.d[pa[k]], V = sd.d[pb[k]];
      float* w4 = T + tab::W4 + 5 * k;
      w4[0] = (float)(0.25 * U.xx * V.xx);
      w4[1] = (float)(0.5 * (U.xx * V.xy + U.xy * V.xx));
      w4[2] = (float)(0.25 * (U.xx * V.yy + 4.0 * U.xy * V.xy + U.yy * V.xx));
      w4[3] = (float)(0.5 * (U.xy * V.yy + U.yy * V.xy));
      w4[4] = (float)(0.25 * U.yy * V.yy);
      T[tab::W2 + 3 * k + 0] = (float)(0.5 * sd.dd[k].xx);
      T[tab::W2 + 3 * k + 1] = (float)(sd.dd[k].xy);
      T[tab::W2 + 3 * k + 2] = (float)(0.5 * sd.dd[k].yy);
    }
  }
  if (t < im.n_psf) {
    const double* ps = im.psf[t];
    float* rec = T + tab::STAR + t * tab::STAR_REC;
    write_gaussian(rec, ps[0], Sym2{ps[3], ps[4], ps[5]});
    rec[tab::S_XIX] = (float)ps[1];
    rec[tab::S_XIY] = (float)ps[2];
  }
  const int n_gal = im.n_psf * ncomp;
  float* G = T + tab::gal_at(n_gal);
  for (int c = t; c < n_gal; c += blockDim.x) {
    const int k = c / ncomp, j = c - k * ncomp;
    const double* ps = im.psf[k];
    const double nu = prof.var[j];
    Sym2 C = {nu * sd.W.xx + ps[3], nu * sd.W.xy + ps[4], nu * sd.W.yy + ps[5]};
    if constexpr (DERIVS)
      write_galaxy(T + tab::EXPO + c * tab::EXPO_REC, G + c * tab::GAL_REC, ps[0] * prof.amp[j], C, nu);
    else
      write_exponent(T + tab::EXPO + c * tab::EXPO_REC, ps[0] * prof.amp[j], C);
  }
}

template <int BLOCK>
__device__ inline double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) sh[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < BLOCK / 64; ++k) r += sh[k];
  return r;
}

// log n! for the integer counts below LFACT_N, filled with the device's own lgamma(n + 1).
__global__ __launch_bounds__(256) void k_lfact(double* __restrict__ t) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < LFACT_N) t[i] = lgamma((double)i + 1.0);
}

// Index of a count's log x! in the table, or -1 where it has none (a fractional, large, negative or
// non-finite value).
__device__ __forceinline__ int table_index(float x) {
  const int n = (int)x;   // truncated
  return (float)n == x && (unsigned)n < (unsigned)LFACT_N ? n : -1;
}

// log x! = log Gamma(z), z = x + 1, of a finite value x >= 0 that the table does not hold; the library's lgamma, which
// also serves negative arguments, takes three times the registers.  From z = 16 on Stirling's series
// (Abramowitz & Stegun 6.1.41; its first term left out, 691 / 360360 z^-11, is 1.1e-16 there); below, the series about 2
// (6.1.33: log Gamma(2 + f) = (1 - gamma) f + sum over k >= 2 of (-1)^k (zeta(k) - 1) f^k / k, kLog2f its
// coefficients from k = 2 on) at |f| <= 1/2 and the recurrence.  Error against 80 bits, rms: 9.3e-16
// for x in 1..15 (the C library's 1.5e-15), 1.8e-14 in 15..100 (2.1e-14), 2.3e-13 in 100..1,000 (2.8e-13), below
// 2e-17 from 0 to 1.5.
__device__ __constant__ double kLog2f[] = {
    0.3224670334241132, -0.0673523010531981, 0.020580808427784546, -0.007385551028673986, 0.0028905103307415234,
    -0.001192753911703261, 0.0005096695247430425, -0.00022315475845357939, 9.945751278180853e-05,
    -4.492623673813314e-05, 2.050721277567069e-05, -9.439488275268397e-06, 4.374866789907488e-06,
    -2.039215753801366e-06, 9.55141213040742e-07, -4.492469198764566e-07, 2.1207184805554665e-07,
    -1.0043224823968099e-07, 4.7698101693639804e-08, -2.2711094608943164e-08, 1.0838659214896955e-08,
    -5.183475041970047e-09, 2.4836745438024785e-09, -1.1921401405860912e-09, 5.731367241678862e-10,
    -2.7595228851242334e-10};
__device__ __noinline__ double log_factorial(float x) {
  const double z = (double)x + 1.0;
  if (z < 16.0) {
    const bool low = z < 1.5;
    const double m = low ? -1.0 : rint(z) - 2.0, f = z - (m + 2.0);
    double p = z, y = z;   // low: Gamma(z) = Gamma(z + 1) / z; otherwise (z - 1) ... (z - m) Gamma(z - m)
    if (!low) p = 1.0;
    for (int i = 0; i < 14 && i < (int)m; ++i) {
      y -= 1.0;
      p *= y;
    }
    constexpr int K = sizeof(kLog2f) / sizeof(double);
    double q = kLog2f[K - 1];
#pragma unroll 1   // (unrolled, the coefficients are held in registers across the pixels: 111 spills)
    for (int k = K - 2; k >= 0; --k) q = fma(q, f, kLog2f[k]);
    const double v = f * fma(f, q, 0.4227843350984671), l = log(p);
    return low ? v - l : v + l;
  }
  const double r = 1.0 / z, r2 = r * r;
  const double series =
      r * fma(r2, fma(r2, fma(r2, fma(r2, 1.0 / 1188.0, -1.0 / 1680.0), 1.0 / 1260.0), -1.0 / 360.0), 1.0 / 12.0);
  return fma(z - 0.5, log(z) - 1.0, series + 0.41893853320467274);   // (z - 1/2) log z - z + log(2 pi) / 2 + series
}

// The host's conditions on a source's estimate (the C entry's check of theta).
__device__ __forceinline__ bool theta_in_range(const double* __restrict__ th) {
  bool ok = true;
  for (int i = 0; i < NP; ++i) ok = ok && fabs(th[i]) < INFINITY;   // false for NaN
  ok = ok && th[2] > 0.0 && th[2] < 1.0 && th[3] >= 0.0 && th[3] <= 1.0 && th[4] > 0.0 && th[4] <= 1.0 && th[6] > 0.0 &&
       th[9] > 0.0 && th[10] > 0.0;
  for (int i = 19; i < NP; ++i) ok = ok && th[i] > 0.0;
  return ok;
}

// One pass over every pixel of an image (one block per image): flags any negative or
// non-finite pixel / neighbour value, and sums the theta-independent part of the pixel term,
// x log E_bg - E_bg - log x!, E_bg = sky + neighbour mean.  log x! of an integer count below
// LFACT_N is read from the table (the same value lgamma gives); without neighbour arrays E_bg
// is the sky at every pixel, so the first two terms are log(sky) sum x - n sky.
//
// An image of the usual sizes is one or two passes of the block, so the loads of a pass are issued
// together: rows that follow each other without gaps are read as one run of 16-byte pieces (4,096 px at
// once; 1,024 px and their neighbour arrays), which need the 4-byte alignment of the pixels only; others pixel by
// pixel, their row and column carried along instead of divided out.  Pixels that are no count of the
// table (calibrated images: every one) are left to a second pass over the image, taken only where there is one.
// It reads the pixels in the same pieces and adds their log x!.  The registers allow eight waves per SIMD; log_factorial
// is called, since inlined its registers came on top of the main pass's (counts in rows with gaps: 53 us).
// 3.6e8 px of 4,000 uneven sources: 436 us; 1,950 us with 4 pixels per thread in flight, a division each
// and lgamma in the loop; 310 us at the rate of a large copy.  1.4e8 px with neighbour arrays: 507 us (1,580).
// 1.8e7 px of 2,000 sources, counts 32 us (110 before the second pass was split off), fractional values 108 (199;
// 369 with the library's lgamma there, a division a pixel and one load in flight); in rows with gaps 37 and
// 247 (109 and 308; 687); with neighbour arrays 81 and 161 (210 and 298; 443).
__global__ __launch_bounds__(256, 8) void k_check_const(const ImgDev* __restrict__ imgs, const double* __restrict__ lfact,
                                                     double* __restrict__ out, int* __restrict__ bad, int n_img,
                                                     const double* __restrict__ theta, int n_src) {
  typedef float V4 __attribute__((ext_vector_type(4), aligned(4)));
  typedef const __attribute__((address_space(1))) V4* GlobalV4;
  __shared__ double sh[4];
  if ((int)blockIdx.x >= n_img) {   // the blocks behind the images': 256 sources' estimates each
    const int s = ((int)blockIdx.x - n_img) * 256 + threadIdx.x;
    if (s < n_src && !theta_in_range(theta + (size_t)s * NP)) atomicOr(bad, FLAG_THETA);
    return;
  }
  const ImgDev& im = imgs[blockIdx.x];
  const int w = im.w, n = im.h * w, pitch = im.pitch, npitch = im.nbr_pitch;
  const GlobalF px = global(im.pix), ne = global(im.nbr_mean), nv = global(im.nbr_var);
  const double sky = im.sky;
  const int t = threadIdx.x;
  double acc = 0.0;      // - log x!, and with neighbour arrays x log E_bg - E_bg
  double sx = 0.0;       // without neighbour arrays: sum of x
  bool rare = false;     // a pixel that is no count of the table
  bool flag = false;     // a pixel or neighbour value out of range
  if (!ne && !nv) {
    auto term = [&](float x, unsigned& sum) {
      const int k = table_index(x);
      rare |= k < 0;
      const int i = max(k, 0);
      acc -= lfact[i];
      sum += (unsigned)i;
    };
    if (pitch == w) {
      constexpr int U = 4;
      const int n4 = n >> 2;
      for (int m0 = t; m0 < n4; m0 += U * 256) {
        V4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = ((GlobalV4)px)[min(m0 + u * 256, n4 - 1)];
        unsigned sum = 0;   // at most 16 counts below LFACT_N
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (m0 + u * 256 >= n4) break;
#pragma unroll
          for (int j = 0; j < 4; ++j) term(x[u][j], sum);
        }
        sx += (double)sum;
      }
      const int m = 4 * n4 + t;   // at most three pixels are left
      if (m < n) {
        unsigned sum = 0;
        term(px[m], sum);
        sx += (double)sum;
      }
    } else {
      constexpr int U = 8;
      const int dr = 256 / w, dc = 256 - dr * w;
      int r = t / w, c = t - r * w;
      for (int m0 = t; m0 < n; m0 += U * 256) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          x[u] = px[m0 + u * 256 < n ? (int64_t)r * pitch + c : 0];
          r += dr;
          c += dc;
          if (c >= w) {
            c -= w;
            ++r;
          }
        }
        unsigned sum = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (m0 + u * 256 >= n) break;
          term(x[u], sum);
        }
        sx += (double)sum;
      }
    }
  } else {
    auto term = [&](float x, float e, float v) {
      const int k = table_index(x);
      rare |= k < 0;
      flag |= !(e >= 0.f) || !(e < INFINITY) || !(v >= 0.f) || !(v < INFINITY);
      const double ebg = sky + (double)e;
      acc += (double)x * log(ebg) - ebg - lfact[max(k, 0)];
    };
    if (pitch == w && npitch == w) {
      const int n4 = n >> 2;
      for (int m = t; m < n4; m += 256) {
        const V4 x = ((GlobalV4)px)[m], e = ne ? ((GlobalV4)ne)[m] : V4{0.f, 0.f, 0.f, 0.f};
        const V4 v = nv ? ((GlobalV4)nv)[m] : V4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) term(x[j], e[j], v[j]);
      }
      const int m = 4 * n4 + t;
      if (m < n) term(px[m], ne ? ne[m] : 0.f, nv ? nv[m] : 0.f);
    } else {
      constexpr int U = 4;
      const int dr = 256 / w, dc = 256 - dr * w;
      int r = t / w, c = t - r * w;
      for (int m0 = t; m0 < n; m0 += U * 256) {
        float x[U], e[U], v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = m0 + u * 256 < n;
          const int64_t o = in ? (int64_t)r * pitch + c : 0, on = in ? (int64_t)r * npitch + c : 0;
          x[u] = px[o];
          e[u] = ne ? ne[on] : 0.f;
          v[u] = nv ? nv[on] : 0.f;
          r += dr;
          c += dc;
          if (c >= w) {
            c -= w;
            ++r;
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (m0 + u * 256 >= n) break;
          term(x[u], e[u], v[u]);
        }
      }
    }
  }
  const bool one_sky = !ne && !nv;
  if (__syncthreads_or(rare)) {
    const auto more = [&](float x) {
      if (table_index(x) >= 0) return;
      const bool ok = x >= 0.f && x < INFINITY;
      flag |= !ok;
      sx += (double)x;   // (with neighbour arrays the main pass has x's other term)
      acc -= log_factorial(ok ? x : 0.f);
    };
    if (pitch == w) {
      const int n4 = n >> 2;
#pragma unroll 1
      for (int m = t; m < n4; m += 256) {
        V4 x = ((GlobalV4)px)[m];
#pragma unroll 1
        for (int j = 0; j < 4; ++j) {
          more(x.x);
          x = V4{x.y, x.z, x.w, x.x};
        }
      }
      const int m = 4 * n4 + t;
      if (m < n) more(px[m]);
    } else {
      const int dr = 256 / w, dc = 256 - dr * w;
      int r = t / w, c = t - r * w;
#pragma unroll 1
      for (int m0 = t; m0 < n; m0 += 4 * 256) {
        V4 x;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[u] = m0 + u * 256 < n ? px[(int64_t)r * pitch + c] : 0.f;
          r += dr;
          c += dc;
          if (c >= w) {
            c -= w;
            ++r;
          }
        }
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
          more(x.x);
          x = V4{x.y, x.z, x.w, x.x};
        }
      }
    }
  }
  if (one_sky) acc += log(sky) * sx;
  const double tot = block_sum<256>(acc, sh);
  if (t == 0) out[blockIdx.x] = one_sky ? tot - (double)n * sky : tot;
  if (flag) atomicOr(bad, FLAG_PIXELS);
}

// Plain start: aperture flux (radius 3 px around the catalog position) in the
// r-band images, prior moments for the rest.  One block per source.
__global__ __launch_bounds__(256) void k_plain_init(const SrcDev* __restrict__ srcs, const ImgDev* __restrict__ imgs,
                                                    PriorDev prior, double* __restrict__ theta) {
  __shared__ double sh[4];
  __shared__ double flux_sum;
  __shared__ int n_r;
  const int s = blockIdx.x;
  double* th = theta + (size_t)s * NP;
  const double ux = th[0], uy = th[1];
  if (threadIdx.x == 0) {
    flux_sum = 0.0;
    n_r = 0;
  }
  __syncthreads();
  for (int i = srcs[s].img_begin; i < srcs[s].img_end; ++i) {
    const ImgDev& im = imgs[i];
    if (im.band != 2) continue;
    const double px = im.wcs[0] * ux + im.wcs[1] * uy + im.wcs[4];
    const double py = im.wcs[2] * ux + im.wcs[3] * uy + im.wcs[5];
    const int n = im.h * im.w;
    double acc = 0.0;
    for (int m = threadIdx.x; m < n; m += 256) {
      const int r = m / im.w, c = m - r * im.w;
      const double dx = im.origin[0] + c - px, dy = im.origin[1] + r - py;
      if (dx * dx + dy * dy <= 9.0) acc += ((double)im.pix[(size_t)r * im.pitch + c] - im.sky) / im.calib;
    }
    const double tot = block_sum<256>(acc, sh);
    if (threadIdx.x == 0) {
      flux_sum += tot;
      n_r += 1;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double f = n_r > 0 ? flux_sum / n_r : 1.0;
    const double r1 = log(fmax(f, 1.0));
    th[2] = 0.5;
    th[3] = 0.5;
    th[4] = 0.7;
    th[5] = 0.0;
    th[6] = 1.5;
    th[7] = r1;
    th[8] = r1;
    th[9] = prior.r_var[0];
    th[10] = prior.r_var[1];
    for (int j = 0; j < 4; ++j) {
      th[11 + j] = prior.c_mean[0][j];
      th[15 + j] = prior.c_mean[1][j];
      th[19 + j] = prior.c_diag[0][j];
      th[23 + j] = prior.c_diag[1][j];
    }
  }
}

}  // namespace

hipError_t launch_setup(const ImgDev* imgs, int n_img, const double* theta, const int* src_flag, ProfDev prof,
                        float* tables, int tstride, hipStream_t st, bool derivs) {
  if (n_img <= 0) return hipSuccess;
  const auto k = derivs ? &k_setup<true> : &k_setup<false>;
  hipLaunchKernelGGL(k, dim3(n_img), dim3(64), 0, st, imgs, theta, src_flag, prof, tables, tstride);
  return hipGetLastError();
}

hipError_t launch_lfact(double* table, hipStream_t st) {
  hipLaunchKernelGGL(k_lfact, dim3((LFACT_N + 255) / 256), dim3(256), 0, st, table);
  return hipGetLastError();
}

hipError_t launch_check_const(const ImgDev* imgs, int n_img, const double* lfact, double* img_const, int* bad,
                              hipStream_t st, const double* theta, int n_src) {
  const auto launch = [&](int ni, int ns) {
    const int blocks = ni + (ns + 255) / 256;
    if (blocks > 0)
      hipLaunchKernelGGL(k_check_const, dim3(blocks), dim3(256), 0, st, imgs, lfact, img_const, bad, ni, theta, ns);
    return hipGetLastError();
  };
  // the estimates by themselves where the launch would otherwise hold 2^32 threads
  if (n_img + (n_src + 255) / 256 < 1 << 24) return launch(n_img, n_src);
  const hipError_t e = launch(n_img, 0);
  return e != hipSuccess ? e : launch(0, n_src);
}

hipError_t launch_check_theta(const double* theta, int n_src, int* bad, hipStream_t st) {
  if (n_src <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_check_const, dim3((n_src + 255) / 256), dim3(256), 0, st, nullptr, nullptr, nullptr, bad, 0, theta,
                     n_src);
  return hipGetLastError();
}

hipError_t launch_plain_init(const SrcDev* srcs, int n_src, const ImgDev* imgs, PriorDev prior, double* theta,
                             hipStream_t s) {
  if (n_src <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plain_init, dim3(n_src), dim3(256), 0, s, srcs, imgs, prior, theta);
  return hipGetLastError();
}

}  // namespace celeste
