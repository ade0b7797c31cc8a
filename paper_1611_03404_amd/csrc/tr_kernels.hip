// Trust-region Newton state machine on the device (section III-B: Newton's method
// with updates constrained by a trust region, dense hand-derived Hessian, per
// source).  A block of four wavefronts per active source solves the 27x27 FP64 subproblem
//     maximise g'p + p'Hp/2  subject to |p| <= Delta     (unconstrained coordinates)
// through a cyclic Jacobi eigendecomposition of B = -H (parallel round-robin
// ordering, 14 disjoint rotations per round, applied to B in LDS by 2x2 blocks and to the
// eigenvectors in registers while the next round's are formed, one barrier a round), followed by the secular
// equation |(B + sI)^{-1} g| = Delta solved by safeguarded Newton on 1/|p(s)|
// (More-Sorensen), including the hard case.  Where B is positive definite, Cholesky
// factorisations of B + lam I give the step instead (the interior Newton step, or the
// boundary step by Newton's method on lam).  A separate kernel applies the
// ratio test, updates the radius and takes an accepted step over, one wavefront per source.
#include <math.h>

#include "celeste_internal.h"
#include "psi_map.h"
#include "wave.h"

namespace celeste {

namespace {

constexpr int NPAD = 28;   // 27 padded to an even order for the round-robin schedule

// ---------------------------------------------------------------- start of a fit
__global__ void k_fit_init(FitDev st, int n_src, FitParams fp) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_src) return;
  double* th = st.theta + (size_t)s * NP;
  double* ps = st.psi + (size_t)s * NP;
  double* u0 = st.u0 + 2 * s;
  u0[0] = th[0];
  u0[1] = th[1];
  for (int i = 0; i < NP; ++i) {
    const Box b = box_of(i, u0, fp.u_box);
    ps[i] = to_psi1(th[i], b);
    double d1, d2;
    th[i] = to_theta1(ps[i], b, &d1, &d2);
  }
  double* V = st.V + (size_t)s * NP * NP;
  for (int i = 0; i < NP * NP; ++i) V[i] = (i % (NP + 1) == 0) ? 1.0 : 0.0;
  st.delta[s] = fp.delta0;
  st.iter[s] = 0;
  st.status[s] = CELESTE_MAX_ITER;
  st.active[s] = 1;
  st.need_full[s] = 1;
  st.n_full[s] = 0;
  st.n_acc[s] = 0;
  st.pred[s] = 0.0;
  st.samp[s] = 0;
  st.sw[s] = 0;
}

// Surrogate start: theta = T(psi) with the position box centred on the catalog position.
__global__ void k_psi_to_theta(const float* __restrict__ psi, const double* __restrict__ theta_cat,
                               double* __restrict__ theta_out, int n_src, double u_box) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_src) return;
  const double u0[2] = {theta_cat[(size_t)s * NP], theta_cat[(size_t)s * NP + 1]};
  for (int i = 0; i < NP; ++i) {
    double d1, d2;
    theta_out[(size_t)s * NP + i] = to_theta1((double)psi[(size_t)s * NP + i], box_of(i, u0, u_box), &d1, &d2);
  }
}

// Keep the surrogate start (theta_trial, ELBO f_trial) where its ELBO is finite and higher
// than the plain start's (theta, f); otherwise flag the fallback.
__global__ void k_choose_start(FitDev st, int n_src) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_src) return;
  const double fs = st.f_trial[s], fp = st.f[s];
  if (isfinite(fs) && (!isfinite(fp) || fs > fp)) {
    for (int i = 0; i < NP; ++i) st.theta[(size_t)s * NP + i] = st.theta_trial[(size_t)s * NP + i];
    st.f[s] = fs;
    st.flags[s] = 0;
  } else {
    st.flags[s] = CELESTE_FLAG_FALLBACK_USED;
  }
}

// A source whose starting ELBO is not finite is not fitted.
__global__ void k_fit_start(FitDev st, int n_src) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_src) return;
  if (!isfinite(st.f[s])) {
    st.status[s] = CELESTE_NONFINITE;
    st.active[s] = 0;
    st.need_full[s] = 0;
  }
}

// The circle method over NPAD players (player M = NPAD - 1 fixed, the rest rotating): pair k of round r
// is (M, r) for k = 0 and (r + k, r - k) mod M otherwise.
constexpr unsigned PM = NPAD - 1;
__device__ __forceinline__ unsigned wrap(unsigned x) { return min(x, x - PM); }          // x in [0, 2 PM)
__device__ __forceinline__ unsigned player_u(unsigned r, unsigned k) { return k == 0 ? PM : wrap(r + k); }
__device__ __forceinline__ unsigned player_v(unsigned r, unsigned k) { return wrap(r + (k == 0 ? 0 : PM - k)); }

// Where the lane of pair k of round r finds what its rotation needs, for r > 0 in the copy of B before round
// r - 1: pair k joins one player of pair a and one of pair b of that round (a < b), so its entry is one
// element of that 2x2 block after it.  x: the block's four entries (flat indices), p and q: the pair.
// Round 0 reads its pivots from B.
struct NextPivot {
  unsigned short x00, x01, x10, x11;
  unsigned char p, q, a, b, row_q, col_q, pad[2];
};
struct NextPivots {
  NextPivot e[NPAD - 1][NPAD / 2];
  unsigned first_u[NPAD - 1];
};
constexpr NextPivots make_next_pivots() {
  NextPivots t{};
  const int M = NPAD - 1;
  for (int r = 0; r < M; ++r)
    for (int k = 0; k < NPAD / 2; ++k) {
      const int u = k == 0 ? M : (r + k) % M, v = k == 0 ? r : (r + M - k) % M;
      NextPivot& e = t.e[r][k];
      e.p = (unsigned char)(u < v ? u : v);
      e.q = (unsigned char)(u < v ? v : u);
      if (r == 0) continue;
      // the pairs of round r - 1 that hold players u and v
      int pair[2] = {0, 0};
      for (int w = 0; w < 2; ++w) {
        const int x = w == 0 ? u : v, d = (x - (r - 1) + M) % M;
        pair[w] = x == M || d == 0 ? 0 : (d <= M / 2 ? d : M - d);
      }
      const int first = pair[0] < pair[1] ? 0 : 1;
      const int a = pair[first], b = pair[1 - first], row = first == 0 ? u : v, col = first == 0 ? v : u;
      int lo[2] = {0, 0}, hi[2] = {0, 0};
      for (int w = 0; w < 2; ++w) {
        const int k2 = w == 0 ? a : b;
        const int u2 = k2 == 0 ? M : (r - 1 + k2) % M, v2 = k2 == 0 ? r - 1 : (r - 1 + M - k2) % M;
        lo[w] = u2 < v2 ? u2 : v2;
        hi[w] = u2 < v2 ? v2 : u2;
      }
      e.a = (unsigned char)a;
      e.b = (unsigned char)b;
      e.row_q = row == hi[0];
      e.col_q = col == hi[1];
      int x[4] = {0, 0, 0, 0};
      for (int w = 0; w < 4; ++w) {
        const int i = w < 2 ? lo[0] : hi[0], j = w % 2 == 0 ? lo[1] : hi[1];
        x[w] = (i < j ? i : j) * (NPAD + 1) + (i < j ? j : i);
      }
      e.x00 = (unsigned short)x[0];
      e.x01 = (unsigned short)x[1];
      e.x10 = (unsigned short)x[2];
      e.x11 = (unsigned short)x[3];
    }
  // bit k of first_u[r]: the first player of pair k is the smaller one
  for (int r = 0; r < M; ++r)
    for (int k = 1; k < NPAD / 2; ++k)
      if ((r + k) % M < (r + M - k) % M) t.first_u[r] |= 1u << k;
  return t;
}
__device__ const NextPivots kNextPivots = make_next_pivots();

// A rotation of the plane (p, q): the entries of a row (or column) pair after it.  Written out so that
// every use rounds alike.
__device__ __forceinline__ double rot_p(double c, double sn, double xp, double xq) { return fma(c, xp, -(sn * xq)); }
__device__ __forceinline__ double rot_q(double c, double sn, double xp, double xq) { return fma(sn, xp, c * xq); }

// flat index of (i, j) in the LDS matrices
constexpr int LDP = NPAD + 1;
__device__ __forceinline__ int at(int i, int j) { return (int)__umul24((unsigned)i, (unsigned)LDP) + j; }
// ... of (i, j) in the upper triangle
__device__ __forceinline__ int upper(int i, int j) { return at(min(i, j), max(i, j)); }

// The trust-region subproblem of one source: one block of four wavefronts.  A solve is a chain of short
// dependent steps (27 rounds a Jacobi sweep, 27 columns a factorisation), so its time is their latency
// and, with a few hundred sources or fewer, the launch's time is one solve's.  The work of a step is
// spread over the wavefronts, and in a Jacobi round the one long chain (three divisions and two square
// roots per rotation) runs ahead of the rest: wavefront 0 forms the next round's rotations from
// the few entries they need, which it rotates itself, while 1 and 2 rotate B's upper triangle by this
// round's (from one LDS copy into the other) and 3 rotates V, a row per lane in registers: one barrier a
// round, each wavefront in its own loop so that only V's holds V's registers.  (V in LDS took over
// half of a round's LDS accesses, which bound large launches: 12,000 sources' fits spent 32.5 ms here.)
// Sums over the wavefront stay in the vector unit; triangular solves keep their vector in the lanes of
// one wavefront.  Every entry of B, V and the factors sees the operations of a one-wavefront solve in the
// same order.  One source, mean of 23 solves: 68 us (138 us on one wavefront); slowest of 1,000 sources,
// mean of 48 launches: 126 us (229 us); fits of 12,000 sources: 21.4 ms in all (26.8 ms);
// registers held to six waves per SIMD (three otherwise, and 26.2 ms).
constexpr int TRT = 256;

__global__ __launch_bounds__(TRT, 6) void k_tr(FitDev st, FitParams fp) {
  __shared__ double Bm[2][NPAD * LDP];   // B; the Jacobi rounds go from one to the other
  __shared__ double V[NPAD][LDP];        // eigenvectors; the Cholesky paths' factor before that
  double (*B)[LDP] = reinterpret_cast<double (*)[LDP]>(Bm[0]);
  __shared__ double g[NPAD], gt[NPAD], pt[NPAD], pst[NPAD], y[NPAD], d1s[NP], d2s[NP];
  __shared__ double2 rcs[2][NPAD / 2];   // (cos, sin) of a round's rotations, of this round and the next
  __shared__ double rtt[2][NPAD / 2];    // tangents, 0 where there is no rotation
  __shared__ double dg[NPAD];            // wavefront 0: diagonal of B
  __shared__ double red[2][TRT / 64];
  __shared__ double s_a, s_b;
  __shared__ int s_curv, done;
  const int s = blockIdx.x;
  if (s == 0 && threadIdx.x == 0) *st.n_active = 0;   // k_accept counts into it
  if (!st.active[s]) return;
  const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  if (t == 0 && st.need_full[s]) {
    st.n_full[s] += 1;
    st.need_full[s] = 0;
  }
  const double* ps = st.psi + (size_t)s * NP;
  const double* gn = st.g + (size_t)s * NP;
  const double* Hn = st.H + (size_t)s * NP * NP;
  const double* u0 = st.u0 + 2 * s;
  // transform to unconstrained coordinates: g = t' g_n, B = -(D H D + diag(t'' g_n))
  if (t < NP) {
    double d1, d2;
    to_theta1(ps[t], box_of(t, u0, fp.u_box), &d1, &d2);
    d1s[t] = d1;
    d2s[t] = d2;
  }
  __syncthreads();
  for (int k = t; k < NPAD * NPAD; k += TRT) {
    const int i = k / NPAD, j = k - i * NPAD;
    double b = 0.0;
    if (i < NP && j < NP) {
      b = -d1s[i] * Hn[i * NP + j] * d1s[j];
      if (i == j) b -= d2s[i] * gn[i];
    }
    B[i][j] = b;
  }
  if (t < NPAD) g[t] = t < NP ? d1s[t] * gn[t] : 0.0;
  __syncthreads();
  const double delta = st.delta[s];
  // the step goes to pst, its predicted gain to pred (thread 0), whether B is positive semi-definite to
  // the curvature tolerance to s_curv
  double pred = 0.0;
  if (t == 0) s_curv = 1;

  // ---- Cholesky paths.  Where B is positive definite, the subproblem's solution is
  // p(lam) = (B + lam I)^{-1} g with lam = 0 if |p(0)| <= Delta (the interior Newton step), and
  // otherwise the lam > 0 with |p(lam)| = Delta (optimality conditions of Nocedal & Wright,
  // Theorem 4.1).  That lam is found by Newton's method on 1/|p(lam)| - 1/Delta from lam = 0
  // (Nocedal & Wright, Algorithm 4.3, with q = L^{-1} p): the function is concave and increasing
  // for lam >= 0, so the iterates increase to the root and B + lam I stays positive definite.
  // Each step costs one Cholesky factorisation (right-looking in LDS, one column per step, the
  // forward substitution carried along) and two triangular solves, instead of the
  // eigendecomposition.  B indefinite or nearly singular (a pivot at most 1e-12 of the largest
  // diagonal entry), or a boundary step not within 1e-9 Delta of the radius after 30 Newton
  // steps, takes the eigendecomposition below.
  int path = 2;   // 0: interior step by Cholesky, 1: boundary step by Cholesky, 2: eigendecomposition
  if (fp.tr_chol) {
    double dmax = lane < NP ? B[lane][lane] : -INFINITY;   // the same on every wavefront
    for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
    dmax = wave_uniform(dmax);
    // V <- the Cholesky factor L of B + lam I (lower triangle), pst <- (B + lam I)^{-1} g and its
    // squared norm (V holds the eigenvectors only in the eigendecomposition path, which loads them afresh).
    // All threads; the decisions are made on values that every thread reads.
    const int cj = t & 31, ch = t >> 5;   // trailing update: column cj, rows cj + ch, cj + ch + 8, ...
    auto factor_solve = [&](double lam, double* pn2) -> bool {
      for (int k = t; k < NP * NP; k += TRT) {
        const int i = k / NP, j = k - i * NP;
        V[i][j] = B[i][j] + (i == j ? lam : 0.0);
      }
      if (t < NPAD) y[t] = g[t];
      __syncthreads();
#pragma unroll 1
      for (int k = 0; k < NP; ++k) {
        const double piv = V[k][k];   // the same value on every thread: the decision is uniform
        if (!(piv > 1e-12 * (dmax + lam))) {
          __syncthreads();
          return false;
        }
        const double lkk = sqrt(piv);
        // (V[k][k] is read above by every thread and written only after the barrier)
        if (t > k && t < NP) V[t][k] /= lkk;
        if (t == k) y[k] /= lkk;
        __syncthreads();
        if (cj > k && cj < NP && ch < 8) {
          const double ljk = V[cj][k];
          double a[4], l[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int i = min(cj + ch + 8 * u, NP - 1);
            l[u] = V[i][k];
            a[u] = V[i][cj];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int i = cj + ch + 8 * u;
            if (i < NP) V[i][cj] = a[u] - l[u] * ljk;
          }
        }
        if (t > k && t < NP) y[t] -= V[t][k] * y[k];
        if (t == k) V[k][k] = lkk;
        __syncthreads();
      }
      // back substitution L' p = y, one unknown per step, lane k of wavefront 0 keeping p_k
      if (wv == 0) {
        double yt = lane < NP ? y[lane] : 0.0, pk = 0.0;
        const double dt = lane < NP ? V[lane][lane] : 1.0;
        double row = V[NP - 1][min(lane, NP - 1)];
#pragma unroll 1
        for (int k = NP - 1; k >= 0; --k) {
          const double cur = row;
          row = V[max(k - 1, 0)][min(lane, NP - 1)];
          const double yk = lane_value(yt, k) / lane_value(dt, k);
          if (lane == k) pk = yk;
          if (lane < k) yt -= cur * yk;
        }
        if (lane < NP) pst[lane] = pk;
        const double n2 = wave_sum(lane < NP ? pk * pk : 0.0);
        if (lane == 0) s_a = n2;
      }
      __syncthreads();
      *pn2 = s_a;
      return true;
    };
    double pn2 = 0.0, lam = 0.0;
    bool first = true;
    int it = 0;
#pragma unroll 1
    while (dmax > 0.0 && factor_solve(lam, &pn2)) {
      if (first && pn2 <= delta * delta) {
        path = 0;
        break;
      }
      it += first ? 0 : 1;
      first = false;
      if (it >= 30) break;
      const double pn = sqrt(pn2);
      if (fabs(pn - delta) <= 1e-9 * delta) {
        path = 1;
        break;
      }
      // q = L^{-1} p by forward substitution, lane k of wavefront 0 keeping q_k
      if (wv == 0) {
        double yt = lane < NP ? pst[lane] : 0.0, qk = 0.0;
        const double dt = lane < NP ? V[lane][lane] : 1.0;
        double col = V[min(lane, NP - 1)][0];
#pragma unroll 1
        for (int k = 0; k < NP; ++k) {
          const double cur = col;
          col = V[min(lane, NP - 1)][min(k + 1, NP - 1)];
          const double yk = lane_value(yt, k) / lane_value(dt, k);
          if (lane == k) qk = yk;
          if (lane > k && lane < NP) yt -= cur * yk;
        }
        const double n2 = wave_sum(qk * qk);
        if (lane == 0) s_b = n2;
      }
      __syncthreads();
      const double qn2 = s_b;
      lam += (pn2 / qn2) * (pn - delta) / delta;
      if (!(lam >= 0.0)) lam = 0.0;   // only by rounding: |p(0)| > Delta
    }
    if (t == 0 && !first && fp.tr_ctr) atomicAdd(fp.tr_ctr + 5, (unsigned long long)it);
    if (path != 2 && wv == 0) {
      // predicted gain: g'p / 2 inside, g'p - p'Bp/2 with (B + lam I) p = g on the boundary
      const double gp = wave_sum(lane < NP ? g[lane] * pst[lane] : 0.0);
      pred = path == 0 ? 0.5 * gp : 0.5 * (gp + lam * pn2);
    }
    __syncthreads();
  }

  if (path == 2) {
  // warm start: the eigenvectors of the previous model (identity at the first iteration)
  for (int k = t; k < NPAD * NPAD; k += TRT) {
    const int i = k / NPAD, j = k - i * NPAD;
    V[i][j] = (i < NP && j < NP) ? st.V[(size_t)s * NP * NP + i * NP + j] : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  // B <- V^T B V, nearly diagonal when the model changed little since the previous iteration;
  // the Jacobi rotations below accumulate into V, so V ends as the eigenvectors of the model.
  // Thread (h, j) = (t / 32, t % 32), h < 7, j < NPAD, forms column j of each product for rows 4 h ..
  // 4 h + 3 in registers (one LDS read of its own column and broadcast reads of the other operand per
  // r; every entry summed over r in increasing order) and stores them after the barrier.
  {
    constexpr int HR = 4;
    const int cj = t & 31, r0 = (t >> 5) * HR;
    const bool cl = cj < NPAD && r0 < NPAD;
    double acc[HR];
#pragma unroll
    for (int i = 0; i < HR; ++i) acc[i] = 0.0;
    if (cl)
#pragma unroll 4
      for (int r = 0; r < NPAD; ++r) {
        const double v = V[r][cj];
#pragma unroll
        for (int i = 0; i < HR; ++i) acc[i] += B[r0 + i][r] * v;
      }
    __syncthreads();
    if (cl)
#pragma unroll
      for (int i = 0; i < HR; ++i) B[r0 + i][cj] = acc[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HR; ++i) acc[i] = 0.0;
    if (cl)
#pragma unroll 4
      for (int r = 0; r < NPAD; ++r) {
        const double b = B[r][cj];
#pragma unroll
        for (int i = 0; i < HR; ++i) acc[i] += V[r][r0 + i] * b;
      }
    __syncthreads();
    if (cl)
#pragma unroll
      for (int i = 0; i < HR; ++i) B[r0 + i][cj] = acc[i];
    __syncthreads();
  }
  // symmetrise (the Hessian is assembled symmetrically; this removes rounding asymmetry)
  for (int k = t; k < NPAD * NPAD; k += TRT) {
    const int i = k / NPAD, j = k - i * NPAD;
    if (i < j) {
      const double m = 0.5 * (B[i][j] + B[j][i]);
      B[i][j] = m;
      B[j][i] = m;
    }
  }
  __syncthreads();

  // ---- cyclic Jacobi, round-robin parallel ordering
  constexpr int NPR = NPAD / 2;                     // disjoint rotations per round
  constexpr int NBLK = NPR * (NPR - 1) / 2;         // off-diagonal 2x2 blocks of B per round (91)
  // wavefronts 1 and 2: one block of B each thread, an off-diagonal one (pairs a < b) or a pair's own
  int blk_a = -1, blk_b = -1;
  if (wv == 1 || wv == 2) {
    int idx = t - 64, a = 0;
    if (idx < NBLK) {
      while (idx >= NPR - 1 - a) {
        idx -= NPR - 1 - a;
        ++a;
      }
      blk_a = a;
      blk_b = a + 1 + idx;
    } else if (idx < NBLK + NPR) {
      blk_a = blk_b = idx - NBLK;
    }
  }
  auto rotate_b = [&](unsigned r, const double* from, double* to, const double2* cs, const double* tn) {
    const unsigned ua = player_u(r, blk_a), va = player_v(r, blk_a), ub = player_u(r, blk_b), vb = player_v(r, blk_b);
    const int p1 = min(ua, va), q1 = max(ua, va), p2 = min(ub, vb), q2 = max(ub, vb);
    const int i00 = upper(p1, p2), i01 = upper(p1, q2), i10 = upper(q1, p2), i11 = upper(q1, q2);
    const double x00 = from[i00], x01 = from[i01], x10 = from[i10], x11 = from[i11];
    const double2 a = cs[blk_a], b = cs[blk_b];
    if (blk_a != blk_b) {
      // columns first, then rows
      const double y00 = rot_p(b.x, b.y, x00, x01), y01 = rot_q(b.x, b.y, x00, x01);
      const double y10 = rot_p(b.x, b.y, x10, x11), y11 = rot_q(b.x, b.y, x10, x11);
      to[i00] = rot_p(a.x, a.y, y00, y10);
      to[i01] = rot_p(a.x, a.y, y01, y11);
      to[i10] = rot_q(a.x, a.y, y00, y10);
      to[i11] = rot_q(a.x, a.y, y01, y11);
    } else {
      // a pair's own block takes the rotated eigenvalue estimates and an exact zero
      const double tt = tn[blk_a];
      to[i00] = tt != 0.0 ? fma(-tt, x01, x00) : x00;
      to[i11] = tt != 0.0 ? fma(tt, x01, x11) : x11;
      to[i01] = tt != 0.0 ? 0.0 : x01;
    }
  };
  // one barrier that every wavefront reaches from its own loop
  auto sync = []() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };
  int sweeps = 0, cur = 0;   // cur: the copy of B that holds it
  // whether another sweep is taken (the same on every thread; two barriers)
  auto another = [&]() -> bool {
    double off = 0.0, fro = 0.0;
    for (int k = t; k < NPAD * NPAD; k += TRT) {
      const int i = k / NPAD, j = k - i * NPAD;
      if (i > j) continue;
      const double x = Bm[cur][at(i, j)], v = x * x;
      fro += i == j ? v : 2.0 * v;
      off += i == j ? 0.0 : 2.0 * v;
    }
    off = wave_sum(off);
    fro = wave_sum(fro);
    if (lane == 0) {
      red[0][wv] = off;
      red[1][wv] = fro;
    }
    sync();
    off = fro = 0.0;
#pragma unroll
    for (int w = 0; w < TRT / 64; ++w) {
      off += red[0][w];
      fro += red[1][w];
    }
    sync();
    return sweeps < 40 && !(off <= 1e-30 * fro || fro == 0.0);
  };
  // a sweep is NPAD slots of one barrier each: in slot r wavefront 0 forms round r's rotations (r < NPAD - 1)
  // and the others apply round r - 1's (r > 0)
  if (wv == 0) {
    const int kk = min(lane, NPR - 1);
    for (; another(); ++sweeps) {
      NextPivot np = kNextPivots.e[0][kk];
      for (int r = 0; r < NPAD; ++r) {
        if (r < NPAD - 1 && lane < NPR) {
          const NextPivot e = np;
          np = kNextPivots.e[min(r + 1, NPAD - 2)][kk];   // in flight during this slot
          const double* from = Bm[cur];
          const int p = e.p, q = e.q;
          double apq, app, aqq;
          if (r == 0) {
            apq = from[at(p, q)];
            app = from[at(p, p)];
            aqq = from[at(q, q)];
          } else {
            // the pair's entry after round r - 1, as rotate_b forms it
            const double x00 = from[e.x00], x01 = from[e.x01], x10 = from[e.x10], x11 = from[e.x11];
            const double2 a = rcs[(r - 1) & 1][e.a], b = rcs[(r - 1) & 1][e.b];
            app = dg[p];
            aqq = dg[q];
            const double y0 = e.col_q ? rot_q(b.x, b.y, x00, x01) : rot_p(b.x, b.y, x00, x01);
            const double y1 = e.col_q ? rot_q(b.x, b.y, x10, x11) : rot_p(b.x, b.y, x10, x11);
            apq = e.row_q ? rot_q(a.x, a.y, y0, y1) : rot_p(a.x, a.y, y0, y1);
          }
          // (the test runs beside the chain, whose result a negligible entry's lane drops)
          const bool rotate = (fabs(apq) > 1e-300) & (fabs(apq) > 1e-18 * sqrt(fabs(app * aqq)));
          const double th = (aqq - app) / (2.0 * apq);
          double tt = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
          double c = 1.0 / sqrt(tt * tt + 1.0), sn = tt * c;
          c = rotate ? c : 1.0;
          sn = rotate ? sn : 0.0;
          tt = rotate ? tt : 0.0;
          rcs[r & 1][lane] = make_double2(c, sn);
          rtt[r & 1][lane] = tt;
          dg[p] = tt != 0.0 ? fma(-tt, apq, app) : app;
          dg[q] = tt != 0.0 ? fma(tt, apq, aqq) : aqq;
        }
        sync();
        if (r > 0) cur ^= 1;
      }
    }
  } else if (wv == 3) {
    // lane = row; register j holds the column of player (r + j) mod PM, j < PM, and x[PM] that of player PM: pair
    // k of every round is registers k and PM - k, and a rotation's results go one register down
    const int row = min(lane, NPAD - 1);
    double x[NPAD];
#pragma unroll
    for (int j = 0; j < NPAD; ++j) x[j] = V[row][j];
    for (; another(); ++sweeps)
      for (int r = 0; r < NPAD; ++r) {
        if (r > 0) {
          const double2* cs = rcs[(r - 1) & 1];
          const unsigned first = kNextPivots.first_u[r - 1];
          constexpr int M = NPAD - 1;
          double2 c = cs[0];
          double carry = rot_p(c.x, c.y, x[0], x[M]);   // player M is the larger one; goes to register M - 1
          x[M] = rot_q(c.x, c.y, x[0], x[M]);
#pragma unroll
          for (int k = 1; k < NPR; ++k) {
            c = cs[k];
            const double xu = x[k], xv = x[M - k];
            double nu, nv;
            if ((first >> k) & 1u) {
              nu = rot_p(c.x, c.y, xu, xv);
              nv = rot_q(c.x, c.y, xu, xv);
            } else {
              nu = rot_q(c.x, c.y, xv, xu);
              nv = rot_p(c.x, c.y, xv, xu);
            }
            x[k - 1] = nu;
            x[M - k] = carry;
            carry = nv;
          }
          x[NPR - 1] = carry;   // register M - 1 - (NPR - 1)
        }
        sync();
        if (r > 0) cur ^= 1;
      }
    if (lane < NPAD)
#pragma unroll
      for (int j = 0; j < NPAD; ++j) V[lane][j] = x[j];
  } else {
    for (; another(); ++sweeps)
      for (int r = 0; r < NPAD; ++r) {
        if (r > 0 && blk_a >= 0) rotate_b(r - 1, Bm[cur], Bm[cur ^ 1], rcs[(r - 1) & 1], rtt[(r - 1) & 1]);
        sync();
        if (r > 0) cur ^= 1;
      }
  }
  __syncthreads();
  B = reinterpret_cast<double (*)[LDP]>(Bm[cur]);

  if (t == 0 && fp.tr_ctr) {
    atomicAdd(fp.tr_ctr + 3, (unsigned long long)sweeps);
    if (sweeps == 40) atomicAdd(fp.tr_ctr + 4, 1ull);
  }

  // ---- eigen-coordinates of g; the eigenvectors are kept for the next iteration's start
  if (t < NP) {
    double a = 0.0;
    for (int r = 0; r < NP; ++r) a += V[r][t] * g[r];
    gt[t] = a;
  }
  for (int k = t; k < NP * NP; k += TRT) st.V[(size_t)s * NP * NP + k] = V[k / NP][k % NP];

  // ---- secular equation, one eigen-coordinate per lane of wavefront 0 (lanes >= NP hold neutral values);
  // every reduction is the same on all lanes, so all take the same decisions
  if (wv == 0) {
    const bool on = lane < NP;
    const double li = on ? B[lane][lane] : 0.0, gi = on ? gt[lane] : 0.0;
    auto wsum = [](double x) { return wave_uniform(wave_sum(x)); };
    auto wmin = [](double x) {
      for (int o = 32; o > 0; o >>= 1) x = fmin(x, __shfl_xor(x, o));
      return wave_uniform(x);
    };
    auto wmax = [](double x) {
      for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o));
      return wave_uniform(x);
    };
    const double lam0 = wmin(on ? li : INFINITY);
    // first index holding the smallest eigenvalue
    const unsigned long long at_min = __ballot(on && li == lam0);
    const int i0 = __ffsll((long long)at_min) - 1;
    const double scale = fmax(1.0, wmax(on ? fabs(li) : 0.0));
    const double gn2 = wsum(gi * gi);
    auto pnorm2 = [&](double sv) {
      const double q = on ? gi / (li + sv) : 0.0;
      return wsum(q * q);
    };
    double sv = 0.0, pti = 0.0;
    bool hard = false;
    if (!(lam0 > 1e-14 * scale && pnorm2(0.0) <= delta * delta)) {
      const double slo = fmax(0.0, -lam0);
      const bool bottom = on && fabs(li - lam0) <= 1e-12 * scale;
      const double gbot2 = wsum(bottom ? gi * gi : 0.0);
      const double qrest = (on && !bottom) ? gi / (li + slo) : 0.0;
      const double prest2 = wsum(qrest * qrest);
      if (sqrt(gbot2) <= 1e-12 * fmax(1.0, sqrt(gn2)) && prest2 <= delta * delta) {
        hard = true;
        sv = slo;
        pti = bottom ? 0.0 : qrest;
        if (lane == i0) pti += sqrt(fmax(delta * delta - prest2, 0.0));
      } else {
        double lo = slo, hi = slo + sqrt(gn2) / delta + 1.0;
        sv = (slo > 0.0) ? slo + 1e-12 * scale : 0.0;
        if (pnorm2(sv) > delta * delta) {
          for (int it = 0; it < 200; ++it) {
            const double den = li + sv;
            const double q = on ? gi / den : 0.0;
            const double a2 = wsum(q * q);
            const double b3 = wsum(on ? q * q / den : 0.0);
            const double pn = sqrt(a2);
            if (fabs(pn - delta) <= 1e-13 * delta) break;
            if (pn > delta) lo = fmax(lo, sv); else hi = fmin(hi, sv);
            // Newton on 1/|p(s)| - 1/Delta, kept inside the bracket
            double nx = sv + (a2 / b3) * (pn - delta) / delta;
            if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
            if (nx == sv) break;
            sv = nx;
          }
        }
        // else: |p| <= Delta just above the pole (nearly the hard case): keep sv
      }
    }
    if (!hard) pti = on ? gi / (li + sv) : 0.0;
    if (on) pt[lane] = pti;
    pred = wsum(on ? gi * pti - 0.5 * li * pti * pti : 0.0);
    if (lane == 0) s_curv = lam0 >= -fp.curv_tol * scale ? 1 : 0;
  }
  __syncthreads();
  // the step back in psi coordinates
  if (t < NP) {
    double a = 0.0;
    for (int i = 0; i < NP; ++i) a += V[t][i] * pt[i];
    pst[t] = a;
  }
  }   // eigendecomposition

  if (wv != 0) return;   // the rest is one wavefront's: thread 0's decision, then one coordinate a lane
  if (t == 0) {
    if (fp.tr_ctr) atomicAdd(fp.tr_ctr + path, 1ull);
    // convergence and iteration cap; on the subsampled objective, the switch to the full one
    const double f = st.f[s];
    int d = 0;
    if (st.samp[s]) {
      if (pred <= fp.switch_rtol * fmax(1.0, fabs(f))) {
        st.samp[s] = 0;
        st.sw[s] = 1;
        d = 2;
      } else if (st.iter[s] >= fp.max_iter) {
        st.status[s] = CELESTE_MAX_ITER;
        d = 1;
      }
    } else if (pred <= fp.pred_rtol * fmax(1.0, fabs(f)) && s_curv) {
      st.status[s] = CELESTE_CONVERGED;
      d = 1;
    } else if (st.iter[s] >= fp.max_iter) {
      st.status[s] = CELESTE_MAX_ITER;
      d = 1;
    }
    st.pred[s] = pred;
    if (d == 1) st.active[s] = 0;
    done = d;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (done == 2) {
    // the switch: the trial point is the current point, whose ELBO on the full objective the
    // value pass evaluates (k_accept takes it as the current value)
    if (t < NP) st.theta_trial[(size_t)s * NP + t] = st.theta[(size_t)s * NP + t];
    return;
  }
  if (done) return;
  // ---- step in psi and the trial point
  double* pp = st.p + (size_t)s * NP;
  double* tht = st.theta_trial + (size_t)s * NP;
  double pn2 = 0.0;
  if (t < NP) {
    const double a = pst[t];
    pp[t] = a;
    double d1, d2;
    tht[t] = to_theta1(ps[t] + a, box_of(t, u0, fp.u_box), &d1, &d2);
    pn2 = a * a;
  }
  pn2 = wave_sum(pn2);
  if (t == 0) st.pnorm[s] = sqrt(pn2);
}

// Ratio test, radius update and acceptance; one wavefront per source.  With trial derivatives an accepted step
// takes over the gradient and Hessian evaluated at its trial point, now the current point (a launch of its own for
// that, and a thread per source here: 7.8 + 5.5 us for one source, 14.4 + 4.8 us for 1,000, against
// 5.6 and 7.7 us).
__global__ __launch_bounds__(64) void k_accept(FitDev st, FitParams fp) {
  const int s = blockIdx.x, t = threadIdx.x;
  if (!st.active[s]) return;
  const bool sw = st.sw[s];
  const double ft = st.f_trial[s];
  if (sw) {
    // moved to the full objective: its value at the current point, then its gradient and Hessian
    if (t) return;
    st.sw[s] = 0;
    st.f[s] = ft;
    st.need_full[s] = 1;
    if (!isfinite(ft)) {
      st.status[s] = CELESTE_NONFINITE;
      st.active[s] = 0;
      st.need_full[s] = 0;
      return;
    }
    atomicAdd(st.n_active, 1);
    return;
  }
  const double f = st.f[s], pred = st.pred[s];
  const double rho = isfinite(ft) ? (ft - f) / pred : -INFINITY;
  const double pn = st.pnorm[s];
  double delta = st.delta[s];
  if (rho < 0.25)
    delta = 0.25 * pn;
  else if (rho > 0.75 && pn >= 0.99 * delta)
    delta = fmin(2.0 * delta, fp.delta_max);
  const bool accept = rho > fp.eta, collapsed = delta < fp.delta_min;
  if (accept) {
    const size_t o = (size_t)s * NP;
    if (t < NP) {
      st.psi[o + t] += st.p[o + t];
      st.theta[o + t] = st.theta_trial[o + t];
    }
    if (fp.trial_derivs && !collapsed) {
      if (t < NP) st.g[o + t] = st.g_trial[o + t];
      double v[(NP * NP + 63) / 64];
#pragma unroll
      for (int q = 0; q < (NP * NP + 63) / 64; ++q) v[q] = st.H_trial[o * NP + min(t + 64 * q, NP * NP - 1)];
#pragma unroll
      for (int q = 0; q < (NP * NP + 63) / 64; ++q)
        if (t + 64 * q < NP * NP) st.H[o * NP + t + 64 * q] = v[q];
    }
  }
  if (t) return;
  if (fp.trial_derivs) st.n_full[s] += 1;   // the trial point's value+gradient+Hessian evaluation
  st.delta[s] = delta;
  if (accept) {
    st.f[s] = ft;
    st.need_full[s] = fp.trial_derivs ? 0 : 1;
    st.n_acc[s] += 1;
    if (fp.trial_derivs && fp.taken_px) atomicAdd(fp.taken_px, (unsigned long long)fp.srcs[s].npix);
  }
  st.iter[s] += 1;
  if (collapsed) {
    st.status[s] = CELESTE_TR_COLLAPSED;
    st.active[s] = 0;
    st.need_full[s] = 0;
    return;
  }
  atomicAdd(st.n_active, 1);
}

__global__ void k_fill(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_split(const int* __restrict__ flag, const int* __restrict__ samp, int* __restrict__ fa,
                        int* __restrict__ fb, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int f = flag[i] != 0, sm = samp[i] != 0;
  fa[i] = f && !sm;
  fb[i] = f && sm;
}

__global__ void k_zero(int* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------- linear-response covariance
// Sigma = D (-H_psi)^{-1} D at a fitted theta, H_psi = D H D + diag(D' g) in the fit's
// unconstrained coordinates (D = d theta / d psi, diagonal), one wavefront per source, FP64, a row (then a
// column) per lane in registers: Cholesky factor L of -H_psi (right-looking), L^{-1} by forward
// substitution, and Sigma_psi = L^{-T} L^{-1} summed in the same order for (a, b) and (b, a), so the
// result is exactly symmetric.  status: 0, 1 when a pivot is not positive (-H_psi not positive
// definite), 2 for a non-finite input; cov is NaN where status != 0.
//
// Bound by the chain of 27 pivots' square roots and divisions and by issue: every product's other factor is
// another lane's, read into a scalar register (two lane reads an FP64 multiply-add), with no
// barrier and no LDS access between.  5,000 sources: 65 us (169 us with the matrices in LDS, 729 entries
// over the lanes for each column and a barrier after each part; the Hessians' and covariances' traffic: 12 us).
__global__ __launch_bounds__(64, 4) void k_lr_cov(const double* __restrict__ theta, const double* __restrict__ u0s,
                                                  double u_box, const double* __restrict__ grad,
                                                  const double* __restrict__ hess, double* __restrict__ cov,
                                                  int* __restrict__ status) {
  __shared__ double buf[NP * NP];
  const int s = blockIdx.x, t = threadIdx.x, row = min(t, NP - 1);   // the lanes past the last row repeat it
  const double* H = hess + (size_t)s * NP * NP;
  double* out = cov + (size_t)s * NP * NP;
  for (int k = t; k < NP * NP; k += 64) buf[k] = H[k];
  bool finite_in;
  double d1, d2g;
  {
    const double u0[2] = {u0s[2 * s], u0s[2 * s + 1]}, th = theta[(size_t)s * NP + row], g = grad[(size_t)s * NP + row];
    const Box b = box_of(row, u0, u_box);
    double d2;
    to_theta1(to_psi1(th, b), b, &d1, &d2);
    d2g = d2 * g;
    finite_in = isfinite(th) && isfinite(g) && isfinite(u0[0]) && isfinite(u0[1]);
  }
  asm volatile("" : "+v"(d2g));   // rounded by itself, not fused with the subtraction below
  __syncthreads();
  double m[NP];
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    const double h = 0.5 * (buf[row * NP + c] + buf[c * NP + row]);
    finite_in = finite_in && isfinite(h);
    m[c] = -(d1 * h * lane_value(d1, c));
    asm volatile("" : "+v"(m[c]));
    if (c == row) m[c] -= d2g;
  }
  __syncthreads();
  int bad = __ballot(!finite_in) ? 2 : 0;
  if (!bad) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const double piv = lane_value(m[k], k);
      if (!(piv > 0.0) || !isfinite(piv)) {
        bad = 1;
        break;
      }
      const double lkk = sqrt(piv);
      m[k] = k == row ? lkk : m[k] / lkk;
#pragma unroll
      for (int j = k + 1; j < NP; ++j) m[j] = fma(-m[k], lane_value(m[k], j), m[j]);
    }
  }
  if (bad) {
    for (int k = t; k < NP * NP; k += 64) out[k] = __builtin_nan("");
    if (t == 0) status[s] = bad;
    return;
  }
  double w[NP];   // column `row` of L^{-1}; its entries above the diagonal come out as 0
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    double acc = i == row ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < i; ++k) acc = fma(-lane_value(m[k], i), w[k], acc);
    w[i] = acc / lane_value(m[i], i);
  }
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    double acc = 0.0;
#pragma unroll
    for (int k = b; k < NP; ++k) acc = fma(w[k], lane_value(w[k], b), acc);
    const double v = acc * (d1 * lane_value(d1, b));   // the same rounding for (a, b) and (b, a)
    if (t < NP) buf[t * NP + b] = v;
  }
  __syncthreads();
  for (int k = t; k < NP * NP; k += 64) out[k] = buf[k];
  if (t == 0) status[s] = 0;
}

}  // namespace

hipError_t launch_fit_init(FitDev st, int n_src, FitParams fp, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_init, dim3((n_src + 127) / 128), dim3(128), 0, s, st, n_src, fp);
  return hipGetLastError();
}

hipError_t launch_psi_to_theta(const float* psi, const double* theta_cat, double* theta_out, int n_src,
                               double u_box, hipStream_t s) {
  hipLaunchKernelGGL(k_psi_to_theta, dim3((n_src + 127) / 128), dim3(128), 0, s, psi, theta_cat, theta_out, n_src,
                     u_box);
  return hipGetLastError();
}

hipError_t launch_choose_start(FitDev st, int n_src, hipStream_t s) {
  hipLaunchKernelGGL(k_choose_start, dim3((n_src + 127) / 128), dim3(128), 0, s, st, n_src);
  return hipGetLastError();
}

hipError_t launch_fit_start(FitDev st, int n_src, hipStream_t s) {
  hipLaunchKernelGGL(k_fit_start, dim3((n_src + 127) / 128), dim3(128), 0, s, st, n_src);
  return hipGetLastError();
}

hipError_t launch_tr_step(FitDev st, int n_src, FitParams fp, hipStream_t s) {
  hipLaunchKernelGGL(k_tr, dim3(n_src), dim3(TRT), 0, s, st, fp);
  return hipGetLastError();
}

hipError_t launch_accept(FitDev st, int n_src, FitParams fp, hipStream_t s) {
  hipLaunchKernelGGL(k_accept, dim3(n_src), dim3(64), 0, s, st, fp);
  return hipGetLastError();
}

hipError_t launch_lr_cov(const double* theta, const double* u0, double u_box, const double* grad, const double* hess,
                         int n_src, double* cov, int* status, hipStream_t s) {
  if (n_src <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_lr_cov, dim3(n_src), dim3(64), 0, s, theta, u0, u_box, grad, hess, cov, status);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int n, int value, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill, dim3((n + 255) / 256), dim3(256), 0, s, p, n, value);
  return hipGetLastError();
}

hipError_t launch_split(const int* flag, const int* samp, int* fa, int* fb, int n_src, hipStream_t s) {
  if (n_src <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_split, dim3((n_src + 255) / 256), dim3(256), 0, s, flag, samp, fa, fb, n_src);
  return hipGetLastError();
}

hipError_t launch_zero_int(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero, dim3((n + 127) / 128), dim3(128), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace celeste
