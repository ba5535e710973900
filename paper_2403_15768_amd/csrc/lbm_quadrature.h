// lbm_quadrature.h -- the (q, omega) friction quadrature for gfx950 (part of
// lbm_kernels.hip).
//
//  k_friction_raw   the sum node by node, omega table tiled through LDS, FP64
//                   sums, wavefront + block reduction (few wall nodes)
//  k_friction_full  the same with the screening denominator |1 - g_s g_l e^{-2qd}|^2
//                   and a dispersive liquid mode (complex responses)
//  k_quad_range, k_quad_plan, k_quad_build, k_quad_eval, k_quad_sum
//                   the sum over omega as piecewise polynomials in
//                   Omega sqrt(q d), evaluated per node and q (many wall nodes)
//  k_quad_rest, k_quad_all   node by node, the q points that would need too
//                   many polynomials
//  k_friction_lat   normalisation lambda_k = lambda_target raw_k / raw_ref
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {

// ------------------------------------------------------------ friction quadrature
constexpr int kQuadThreads = 256;
constexpr int kQuadNodes = 4;     // wall nodes per workgroup (share the LDS tile)
constexpr int kQuadTile = 1024;   // omega points per LDS tile

struct OmegaEntry {
  double s, t, v, pad;  // w^2, gamma_s^2 w^2, gamma_s w Im g_l(w) / sinh^2(w/2T)
};

// 1/d for the integrands' denominators (positive, far inside the normal
// range: at least gamma_s^2 (dw/2)^2): the hardware reciprocal refined by
// two Newton-Raphson steps r <- r + r (1 - d r), each of which squares the
// relative error, so the result is within about an ulp of 1/d.  Four fused
// multiply-adds and one reciprocal instead of the scaled, fixed-up IEEE
// division; the sums it feeds hold positive terms, so their relative error
// stays at that level.
__device__ __forceinline__ double recip_nr(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = __builtin_fma(-d, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-d, r, 1.0);
  return __builtin_fma(r, e, r);
}

// raw[k] for k < n uses omega[k]; raw[n] is the reference at omega0.
__global__ void __launch_bounds__(kQuadThreads) k_friction_raw(SpecArgs s,
                                                               const double* __restrict__ omega,
                                                               int64_t n,
                                                               double* __restrict__ raw) {
  __shared__ OmegaEntry tab[kQuadTile];
  __shared__ double red[kQuadNodes][kQuadThreads / 64];
  const int tid = threadIdx.x;
  const int64_t k0 = (int64_t)blockIdx.x * kQuadNodes;
  double om2[kQuadNodes];
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) {
    const int64_t k = k0 + j;
    const double o = k < n ? omega[k] : s.omega0;  // k >= n: reference (k == n) or padding
    om2[j] = o * o;
  }
  const double dq = s.q_max / s.nq, dw = s.w_max / s.nw;
  const double gs2 = s.gamma_s * s.gamma_s, wl2 = s.omega_l * s.omega_l;
  const double gl2 = s.gamma_l * s.gamma_l;
  double acc[kQuadNodes];
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) acc[j] = 0.0;

  for (int b0 = 0; b0 < s.nw; b0 += kQuadTile) {
    const int nb = min(kQuadTile, s.nw - b0);
    __syncthreads();
    for (int b = tid; b < nb; b += kQuadThreads) {
      const double w = ((double)(b0 + b) + 0.5) * dw;
      const double w2 = w * w;
      const double sh = sinh(w / (2.0 * s.T));
      const double dl = wl2 - w2;
      const double iml = s.a_l * wl2 * s.gamma_l * w / (dl * dl + gl2 * w2);
      OmegaEntry e;
      e.s = w2;
      e.t = gs2 * w2;
      e.v = s.gamma_s * w * iml / (sh * sh);
      e.pad = 0.0;
      tab[b] = e;
    }
    __syncthreads();
    for (int ai = tid; ai < s.nq; ai += kQuadThreads) {
      const double q = ((double)ai + 0.5) * dq;
      const double kq = q * q * q * exp(-2.0 * q * s.d);
      const double qd = s.dispersion ? q * s.d : 1.0;
      double P[kQuadNodes], S[kQuadNodes];
#pragma unroll
      for (int j = 0; j < kQuadNodes; j++) {
        P[j] = om2[j] * qd;
        S[j] = 0.0;
      }
      for (int b = 0; b < nb; b++) {
        const OmegaEntry e = tab[b];  // same b for every lane: LDS broadcast
#pragma unroll
        for (int j = 0; j < kQuadNodes; j++) {
          const double dd = P[j] - e.s;
          S[j] = __builtin_fma(e.v, recip_nr(dd * dd + e.t), S[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < kQuadNodes; j++) acc[j] += kq * P[j] * S[j];
    }
  }
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) {
    const double v = wave_sum(acc[j]);
    if (lane == 0) red[j][wv] = v;
  }
  __syncthreads();
  if (tid < kQuadNodes) {
    const int64_t k = k0 + tid;
    if (k <= n) {
      double t = 0;
      for (int w = 0; w < kQuadThreads / 64; w++) t += red[tid][w];
      const double C = 1.0 / (8.0 * M_PI * M_PI * s.T);
      raw[k] = C * dq * dw * t;
    }
  }
}

// The screened form: complex responses g_s = P (d_s + i gamma_s w) / D,
// d_s = P - w^2, D = d_s^2 + gamma_s^2 w^2, and g_l = a_l W (d_l + i gamma_l w)
// / (d_l^2 + gamma_l^2 w^2), W = omega_l^2 + v_l^2 q^2, d_l = W - w^2; with
// z = e^{-2qd} g_s g_l = (e P / D)(a + i b), a = d_s Re g_l - gamma_s w Im g_l,
// b = d_s Im g_l + gamma_s w Re g_l, the term
//   q^3 e^{-2qd} Im g_s Im g_l / (sinh^2 |1 - z|^2)
//   = q^3 e^{-2qd} P (gamma_s w / sinh^2) Im g_l D / ((D - e P a)^2 + (e P b)^2)
// takes one divide (SCREEN = false: the unscreened term with a dispersive
// liquid, q^3 e^{-2qd} P (gamma_s w / sinh^2) Im g_l / D).
constexpr int kFullTile = 512;

struct OmegaEntryFull {
  double w2, gw, t, v, glw, gl2w2, pad0, pad1;  // w^2, gamma_s w, gamma_s^2 w^2,
                                                // gamma_s w / sinh^2, gamma_l w, (gamma_l w)^2
};

template <bool SCREEN>
__global__ void __launch_bounds__(kQuadThreads) k_friction_full(SpecArgs s,
                                                                const double* __restrict__ omega,
                                                                int64_t n,
                                                                double* __restrict__ raw) {
  __shared__ OmegaEntryFull tab[kFullTile];
  __shared__ double red[kQuadNodes][kQuadThreads / 64];
  const int tid = threadIdx.x;
  const int64_t k0 = (int64_t)blockIdx.x * kQuadNodes;
  double om2[kQuadNodes];
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) {
    const int64_t k = k0 + j;
    const double o = k < n ? omega[k] : s.omega0;  // k >= n: reference (k == n) or padding
    om2[j] = o * o;
  }
  const double dq = s.q_max / s.nq, dw = s.w_max / s.nw;
  double acc[kQuadNodes];
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) acc[j] = 0.0;

  for (int b0 = 0; b0 < s.nw; b0 += kFullTile) {
    const int nb = min(kFullTile, s.nw - b0);
    __syncthreads();
    for (int b = tid; b < nb; b += kQuadThreads) {
      const double w = ((double)(b0 + b) + 0.5) * dw;
      const double sh = sinh(w / (2.0 * s.T));
      OmegaEntryFull e;
      e.w2 = w * w;
      e.gw = s.gamma_s * w;
      e.t = e.gw * e.gw;
      e.v = e.gw / (sh * sh);
      e.glw = s.gamma_l * w;
      e.gl2w2 = e.glw * e.glw;
      e.pad0 = e.pad1 = 0.0;
      tab[b] = e;
    }
    __syncthreads();
    for (int ai = tid; ai < s.nq; ai += kQuadThreads) {
      const double q = ((double)ai + 0.5) * dq;
      const double ex = exp(-2.0 * q * s.d);
      const double kq = q * q * q * ex;
      const double qd = s.dispersion ? q * s.d : 1.0;
      const double Wl = s.omega_l * s.omega_l + s.v_l * s.v_l * q * q;
      const double Al = s.a_l * Wl;
      double P[kQuadNodes], eP[kQuadNodes], S[kQuadNodes];
#pragma unroll
      for (int j = 0; j < kQuadNodes; j++) {
        P[j] = om2[j] * qd;
        eP[j] = ex * P[j];
        S[j] = 0.0;
      }
      for (int b = 0; b < nb; b++) {
        const OmegaEntryFull e = tab[b];  // same b for every lane: LDS broadcast
        const double dl = Wl - e.w2;
        const double inv = Al / (dl * dl + e.gl2w2);
        const double Rl = inv * dl, Il = inv * e.glw;
        const double vI = e.v * Il;
        const double c1 = e.gw * Il, c2 = e.gw * Rl;
#pragma unroll
        for (int j = 0; j < kQuadNodes; j++) {
          const double dd = P[j] - e.w2;
          const double D = dd * dd + e.t;
          if constexpr (SCREEN) {
            const double a = dd * Rl - c1, bb = dd * Il + c2;
            const double A = D - eP[j] * a, B = eP[j] * bb;
            S[j] = __builtin_fma(vI * D, recip_nr(A * A + B * B), S[j]);
          } else {
            S[j] = __builtin_fma(vI, recip_nr(D), S[j]);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < kQuadNodes; j++) acc[j] += kq * P[j] * S[j];
    }
  }
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int j = 0; j < kQuadNodes; j++) {
    const double v = wave_sum(acc[j]);
    if (lane == 0) red[j][wv] = v;
  }
  __syncthreads();
  if (tid < kQuadNodes) {
    const int64_t k = k0 + tid;
    if (k <= n) {
      double t = 0;
      for (int w = 0; w < kQuadThreads / 64; w++) t += red[tid][w];
      const double C = 1.0 / (8.0 * M_PI * M_PI * s.T);
      raw[k] = C * dq * dw * t;
    }
  }
}

// ------------------------------------------------------------ piecewise sums
// The sum over omega is a function of one variable per q.  With s = Omega
// sqrt(q d) (s = Omega without dispersion) and P = s^2,
//   Im g_s / |1 - e g_s g_l|^2 = P gamma_s w / |P alpha - beta|^2,
//   alpha = 1 - e g_l (1 unscreened), beta = w^2 + i gamma_s w, e = e^{-2qd},
// so raw = C dq dw sum_q q^3 e P F_q(s),
//   F_q(s) = sum_w v / |s^2 alpha - beta|^2,  v = (gamma_s w / sinh^2) Im g_l:
// every term positive, with poles at +-sqrt(beta / alpha) and their
// conjugates.  The nodes need F_q on [Omega_min, Omega_max] sqrt(q d) only;
// there it is cut into equal panels, each a polynomial of degree
// kTabDeg - 1 through the Chebyshev points.  With every pole at least
// kPoleRatio half-widths from every panel's centre, the ellipse of parameter
// rho = k + sqrt(k^2 - 1) = 8.3 or more around a panel holds no pole.  For a
// pair of poles at the axis, 1 / (k - x)^2, the relative interpolation error
// is at most 2 rho^-20 (1 + 20 (k + 1) / sqrt(k^2 - 1)) = 2e-17 (each term is
// positive, so the terms' relative errors do not add up), below a double's
// rounding.  The same bound keeps the monomial form in the panel's
// own coordinate well conditioned (its coefficients fall like 4.2^-j).
// Without screening and with v_l = 0, F does not depend on q: one table.
//
// Work: 129,024 nodes x 256 q x 20 multiply-adds and a table of up to 256 x
// 256 panels x 20 points x 1024 omegas, instead of 129,024 x 262,144 points.
// Measured (whole lbm_set_friction_spectral and lbm_get_friction): the R = 32
// tube's 129,024 nodes 10.9 -> 0.44 ms, screened 31,744 nodes 5.8 -> 0.30 ms.
// Root mean square error of lambda against long double sums, ten spectra: plain
// 4.1e-16 node by node, 2.6e-16 so; screened 3.1e-16 and 2.4e-16.  The groups of q
// are added from the last to the first: the many beyond the peak of q^3 e^{-2qd}
// while the sum is still small (from the first to the last, each of them
// rounded the whole sum: 3.2e-16 and 5.0e-16).
//
// A table that would need more than kTabCap panels (poles close to the real
// axis, or a wide range of Omega) is not built: its q is summed node by node
// (k_quad_rest; k_quad_all where there is one table for all).
constexpr int kTabDeg = 20;
constexpr int kTabCap = 256;          // panels per table (one per lane of a block at most)
constexpr int kTabGroup = 8;          // q points whose terms are summed first (fixed:
                                      // results do not depend on the scratch)
constexpr double kPoleRatio = 4.2;
constexpr int kRangeBlocks = 64;
constexpr int kBuildPanels = 6;       // panels per block of k_quad_build
constexpr int kBuildTile = 512;       // omega points per LDS tile
constexpr int64_t kTabDoubles = (int64_t)kTabCap * kTabDeg;  // [coefficient][panel]
static_assert(kTabCap <= kQuadThreads, "a block loads one panel per lane");

struct TabInfo {
  double s_lo, inv_h, h;
  int np, pad;  // panels; > kTabCap: no table
};

// one omega point of one q: alpha, beta, v
struct OmegaTerm {
  double ar, ai, br, bi, v;
};

// sqrt(q d) (1 without dispersion) of q point a, rounded the same way
// wherever it is used: Omega sigma is monotonic in Omega, so every node's s
// lies in the planned range
__device__ __forceinline__ double quad_sigma(const SpecArgs& s, int a) {
  const double q = ((double)a + 0.5) * (s.q_max / s.nq);
  return s.dispersion ? sqrt(q * s.d) : 1.0;
}

// the factor of the double sum: dq dw / (8 pi^2 T)
__device__ __forceinline__ double quad_scale(const SpecArgs& s) {
  return 1.0 / (8.0 * M_PI * M_PI * s.T) * (s.q_max / s.nq) * (s.w_max / s.nw);
}

__device__ __forceinline__ OmegaTerm omega_term(const SpecArgs& s, int a, int b) {
  const double q = ((double)a + 0.5) * (s.q_max / s.nq);
  const double w = ((double)b + 0.5) * (s.w_max / s.nw);
  const double sh = sinh(w / (2.0 * s.T));
  const double W = s.omega_l * s.omega_l + s.v_l * s.v_l * q * q;
  const double dl = W - w * w, glw = s.gamma_l * w, gw = s.gamma_s * w;
  const double inv = s.a_l * W / (dl * dl + glw * glw);
  const double Il = inv * glw;
  OmegaTerm t;
  t.ar = 1.0;
  t.ai = 0.0;
  if (s.coupling) {
    const double e = exp(-2.0 * q * s.d);
    t.ar = 1.0 - e * (inv * dl);
    t.ai = -e * Il;
  }
  t.br = w * w;
  t.bi = gw;
  t.v = gw * Il / (sh * sh);
  return t;
}

__device__ __forceinline__ double omega_sum(const OmegaTerm& t, double P, double S) {
  const double X = __builtin_fma(P, t.ar, -t.br), Y = __builtin_fma(P, t.ai, -t.bi);
  return __builtin_fma(t.v, recip_nr(X * X + Y * Y), S);
}

// per-block range of |Omega| over the finite frequencies of the nodes (a bad
// frequency must not spoil the other nodes' tables)
__global__ void __launch_bounds__(kQuadThreads) k_quad_range(const double* __restrict__ omega,
                                                             int64_t n,
                                                             double* __restrict__ range) {
  __shared__ double red[2][kQuadThreads / 64];
  double lo = INFINITY, hi = 0.0;
  for (int64_t k = (int64_t)blockIdx.x * kQuadThreads + threadIdx.x; k < n;
       k += (int64_t)kRangeBlocks * kQuadThreads) {
    const double o = fabs(omega[k]);
    if (o < INFINITY) {
      lo = fmin(lo, o);
      hi = fmax(hi, o);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, o, 64));
    hi = fmax(hi, __shfl_xor(hi, o, 64));
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = lo;
    red[1][threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kQuadThreads / 64; w++) {
      lo = fmin(lo, red[0][w]);
      hi = fmax(hi, red[1][w]);
    }
    range[2 * blockIdx.x] = lo;
    range[2 * blockIdx.x + 1] = hi;
  }
}

// one block per table: the panel width from the poles' distance to the range;
// over (not shared): which q's table would be too long
__global__ void __launch_bounds__(kQuadThreads) k_quad_plan(SpecArgs s, int shared, int a0,
                                                            const double* __restrict__ range,
                                                            TabInfo* __restrict__ info,
                                                            uint8_t* __restrict__ over) {
  __shared__ double red[kQuadThreads / 64];
  double lo = s.omega0, hi = s.omega0;
  for (int b = 0; b < kRangeBlocks; b++) {
    lo = fmin(lo, range[2 * b]);
    hi = fmax(hi, range[2 * b + 1]);
  }
  const int a = shared ? 0 : a0 + (int)blockIdx.x;
  const double s_lo = lo * quad_sigma(s, a), s_hi = hi * quad_sigma(s, shared ? s.nq - 1 : a);
  double d = INFINITY;
  for (int b = threadIdx.x; b < s.nw; b += kQuadThreads) {
    const OmegaTerm t = omega_term(s, a, b);
    const double m = t.ar * t.ar + t.ai * t.ai;
    const double pr = (t.br * t.ar + t.bi * t.ai) / m, pi = (t.bi * t.ar - t.br * t.ai) / m;
    // principal square root, real part >= 0
    const double r = sqrt(pr * pr + pi * pi);
    const double x = sqrt(fmax(0.0, 0.5 * (r + pr))), y = sqrt(fmax(0.0, 0.5 * (r - pr)));
    const double dx = x < s_lo ? s_lo - x : (x > s_hi ? x - s_hi : 0.0);
    const double dist = sqrt(dx * dx + y * y);
    d = dist == dist ? fmin(d, dist) : 0.0;  // alpha = 0 or overflow: no table
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) d = fmin(d, __shfl_xor(d, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kQuadThreads / 64; w++) d = fmin(d, red[w]);
    // panels of at most that width, none beyond the range (there the poles may
    // be closer); a range of one point: a panel around it
    const double widest = 2.0 * d / kPoleRatio, range_s = s_hi - s_lo;
    const double np = ceil(range_s / widest);
    TabInfo t;
    t.np = np <= (double)kTabCap && widest < INFINITY ? max(1, (int)np) : kTabCap + 1;
    t.h = range_s > 0.0 ? range_s / t.np : widest;
    t.inv_h = 1.0 / t.h;
    t.s_lo = range_s > 0.0 ? s_lo : s_lo - 0.5 * t.h;
    t.pad = 0;
    info[blockIdx.x] = t;
    if (!shared) over[a] = t.np > kTabCap;
  }
}

// coefficients of the Chebyshev polynomials T_0 .. T_19 (exact integers)
struct ChebCoef {
  double c[kTabDeg][kTabDeg];
};
constexpr ChebCoef cheb_coef() {
  ChebCoef t{};
  t.c[0][0] = 1.0;
  t.c[1][1] = 1.0;
  for (int k = 2; k < kTabDeg; k++)
    for (int j = 0; j < kTabDeg; j++)
      t.c[k][j] = (j > 0 ? 2.0 * t.c[k - 1][j - 1] : 0.0) - t.c[k - 2][j];
  return t;
}
static __constant__ ChebCoef kCheb = cheb_coef();

// Table points: a block takes kBuildPanels panels (120 points, two per lane
// so that one broadcast read of an omega term serves both), its four waves a
// quarter of the omega points each.  Bound by the FP64 pipe: about 10 issue
// slots per point and omega.
__global__ void __launch_bounds__(kQuadThreads) k_quad_build(SpecArgs s, int shared, int a0,
                                                             const TabInfo* __restrict__ info,
                                                             double* __restrict__ tab) {
  __shared__ OmegaTerm term[kBuildTile];
  __shared__ double part[kQuadThreads / 64][kBuildPanels * kTabDeg];
  __shared__ double cosine[4 * kTabDeg];
  const TabInfo t = info[blockIdx.y];
  const int p0 = (int)blockIdx.x * kBuildPanels;
  if (t.np > kTabCap || p0 >= t.np) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int a = shared ? 0 : a0 + (int)blockIdx.y;
  if (tid < 4 * kTabDeg) cosine[tid] = cospi((double)tid / (2 * kTabDeg));
  __syncthreads();
  constexpr int kHalf = kBuildPanels / 2 * kTabDeg;  // 60 points
  const int pt = lane < kHalf ? lane : 0;
  const int pp = pt / kTabDeg, j = pt - pp * kTabDeg;
  const double xj = 0.5 * cosine[2 * j + 1];
  const double s0 = t.s_lo + ((double)(p0 + pp) + 0.5 + xj) * t.h;
  const double s1 = t.s_lo + ((double)(p0 + kBuildPanels / 2 + pp) + 0.5 + xj) * t.h;
  const double P0 = s0 * s0, P1 = s1 * s1;
  double S0 = 0.0, S1 = 0.0;
  for (int b0 = 0; b0 < s.nw; b0 += kBuildTile) {
    const int nb = min(kBuildTile, s.nw - b0);
    __syncthreads();
    for (int b = tid; b < nb; b += kQuadThreads) term[b] = omega_term(s, a, b0 + b);
    __syncthreads();
    for (int b = wv; b < nb; b += kQuadThreads / 64) {
      const OmegaTerm e = term[b];
      S0 = omega_sum(e, P0, S0);
      S1 = omega_sum(e, P1, S1);
    }
  }
  if (lane < kHalf) {
    part[wv][lane] = S0;
    part[wv][kHalf + lane] = S1;
  }
  __syncthreads();
  constexpr int kPts = kBuildPanels * kTabDeg;
  if (tid < kPts) part[0][tid] = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
  __syncthreads();
  // values at the Chebyshev points -> Chebyshev coefficients -> monomials in
  // the panel's coordinate in [-1, 1]
  const int p = tid / kTabDeg, k = tid - p * kTabDeg;
  if (tid < kPts) {
    double c = 0.0;
    for (int i = 0; i < kTabDeg; i++)
      c += part[0][p * kTabDeg + i] * cosine[(k * (2 * i + 1)) % (4 * kTabDeg)];
    part[1][tid] = c * (k == 0 ? 1.0 / kTabDeg : 2.0 / kTabDeg);
  }
  __syncthreads();
  if (tid < kPts && p0 + p < t.np) {
    double m = 0.0;
    for (int i = kTabDeg - 1 - ((kTabDeg - 1 - k) & 1); i >= k; i -= 2)  // small terms first
      m += part[1][p * kTabDeg + i] * kCheb.c[i][k];
    tab[(int64_t)blockIdx.y * kTabDoubles + k * kTabCap + p0 + p] = m;
  }
}

// One wall node per lane: the sums of q^3 e^{-2qd} P F_q over groups of
// kTabGroup q points.  The q's table sits in LDS, coefficient by coefficient
// (neighbouring nodes have nearly the same Omega, so the panels of a wave are
// few and next to each other: the same place or different banks).  With part,
// block row y takes `per` groups and leaves the sum of each in its row of part;
// without, one block adds all `groups` of them to raw, the last one first, as
// k_quad_sum adds rows.
__global__ void __launch_bounds__(kQuadThreads) k_quad_eval(SpecArgs s, int shared, int g0,
                                                            int groups, int per,
                                                            const double* __restrict__ omega,
                                                            int64_t n,
                                                            const TabInfo* __restrict__ info,
                                                            const double* __restrict__ tab,
                                                            double* __restrict__ part,
                                                            double* __restrict__ raw) {
  __shared__ double lds[kTabDoubles];
  __shared__ double sg[kTabGroup], qd[kTabGroup], wt[kTabGroup];
  if (shared && info[0].np > kTabCap) return;  // left to k_quad_all
  const int tid = threadIdx.x;
  const int64_t k = (int64_t)blockIdx.x * kQuadThreads + tid;
  const double om = fabs(k < n ? omega[k] : s.omega0);  // k >= n: reference or padding
  const bool first = (g0 + groups) * kTabGroup >= s.nq;
  double sum = !part && !first && k <= n ? raw[k] : 0.0;
  for (int gi = 0; gi < per; gi++) {
    // the group within this launch's tables
    const int gl = part ? (int)blockIdx.y * per + gi : groups - 1 - gi;
    if (gl >= groups || gl < 0) break;
    const int ga = (g0 + gl) * kTabGroup;        // its first q point
    const int na = min(kTabGroup, s.nq - ga);
    __syncthreads();
    if (tid < na) {
      const double q = ((double)(ga + tid) + 0.5) * (s.q_max / s.nq);
      sg[tid] = quad_sigma(s, ga + tid);
      qd[tid] = s.dispersion ? q * s.d : 1.0;
      wt[tid] = q * q * q * exp(-2.0 * q * s.d);
    }
    __syncthreads();
    double acc = 0.0;
    for (int i = 0; i < na; i++) {
      const int tb = shared ? 0 : gl * kTabGroup + i;
      const TabInfo t = info[tb];
      if (!shared || (i == 0 && gi == 0)) {
        __syncthreads();
        if (t.np <= kTabCap && tid < t.np) {
          const double* c = tab + (int64_t)tb * kTabDoubles + tid;
#pragma unroll
          for (int m = 0; m < kTabDeg; m++) lds[m * kTabCap + tid] = c[m * kTabCap];
        }
        __syncthreads();
      }
      if (t.np > kTabCap) continue;  // left to k_quad_rest
      const double sv = om * sg[i], P = om * om * qd[i];
      const double u = (sv - t.s_lo) * t.inv_h;
      double F = NAN;  // a node whose frequency is not finite
      if (u >= 0.0 && u < (double)t.np + 0.5) {
        const int p = min((int)u, t.np - 1);
        const double x = 2.0 * (u - (double)p) - 1.0;
        const double* c = lds + p;
        F = c[(kTabDeg - 1) * kTabCap];
#pragma unroll
        for (int m = kTabDeg - 2; m >= 0; m--) F = __builtin_fma(F, x, c[m * kTabCap]);
      }
      acc += wt[i] * P * F;
    }
    sum += acc;
    if (part && k <= n) part[(int64_t)gl * (n + 1) + k] = acc;
  }
  if (!part && k <= n) raw[k] = g0 == 0 ? quad_scale(s) * sum : sum;
}

// raw[k]: the groups' partial sums, the last group first (over several calls
// where the scratch holds fewer groups than there are)
__global__ void __launch_bounds__(kQuadThreads) k_quad_sum(SpecArgs s, int shared, int first,
                                                           int last, int groups,
                                                           const TabInfo* __restrict__ info,
                                                           const double* __restrict__ part,
                                                           int64_t n, double* __restrict__ raw) {
  const int64_t k = (int64_t)blockIdx.x * kQuadThreads + threadIdx.x;
  if (k > n || (shared && info[0].np > kTabCap)) return;
  double t = first ? 0.0 : raw[k];
  for (int g = groups - 1; g >= 0; g--) t += part[(int64_t)g * (n + 1) + k];
  raw[k] = last ? quad_scale(s) * t : t;
}

// The q points without a table (spectra whose omega sum depends on q), node by
// node: adds their sum to raw.  A block takes kRestNodes nodes at a time and
// all its lanes one word of 64 q: lane = (one of the word's points, a part of
// the omegas), so the lanes stay busy whether one point is left over or all of
// them.  Bound by the FP64 pipe: the factors of a (q, omega) pair serve eight
// nodes (with four, 17.2 in place of 15.3 ms below), and the omega table is
// built once per block where it fits.  Before, k_quad_eval summed these points
// one node per lane (bound by its LDS reads, and with few blocks where the
// scratch holds few rows).  256 x 1024 points, screened, every q left over:
// 129,000 nodes 20.3 -> 15.3 ms (k_friction_full 23.0), 18,480 nodes 4.24 ->
// 2.61 ms (3.50); with a dispersive liquid only, 21.0 -> 13.2 ms (15.3).
constexpr int kRestNodes = 8;
constexpr int kRestTile = 1024;

struct RestEntry {
  double w2, gw, v, glw;  // w^2, gamma_s w, gamma_s w / sinh^2, gamma_l w
};

template <bool SCREEN>
__global__ void __launch_bounds__(kQuadThreads)
    k_quad_rest(SpecArgs s, const double* __restrict__ omega, int64_t n,
                const uint8_t* __restrict__ over, double* __restrict__ raw) {
  __shared__ RestEntry tab[kRestTile];
  __shared__ double red[kRestNodes][kQuadThreads / 64];
  __shared__ int pick[64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int any = 0;
  for (int a = tid; a < s.nq; a += kQuadThreads) any |= over[a];
  if (!__syncthreads_or(any)) return;
  const double dq = s.q_max / s.nq, dw = s.w_max / s.nw;
  bool built = false;
  for (int64_t k0 = (int64_t)blockIdx.x * kRestNodes; k0 <= n;
       k0 += (int64_t)gridDim.x * kRestNodes) {
    double om2[kRestNodes], acc[kRestNodes];
#pragma unroll
    for (int j = 0; j < kRestNodes; j++) {
      const int64_t k = k0 + j;
      const double o = k < n ? omega[k] : s.omega0;  // k >= n: reference (k == n) or padding
      om2[j] = o * o;
      acc[j] = 0.0;
    }
    for (int b0 = 0; b0 < s.nw; b0 += kRestTile) {
      const int nb = min(kRestTile, s.nw - b0);
      if (!built) {
        __syncthreads();
        for (int b = tid; b < nb; b += kQuadThreads) {
          const double w = ((double)(b0 + b) + 0.5) * dw;
          const double sh = sinh(w / (2.0 * s.T));
          RestEntry e;
          e.w2 = w * w;
          e.gw = s.gamma_s * w;
          e.v = e.gw / (sh * sh);
          e.glw = s.gamma_l * w;
          tab[b] = e;
        }
        __syncthreads();
        built = s.nw <= kRestTile;
      }
      for (int a0 = 0; a0 < s.nq; a0 += 64) {
        // the word's points, one after the other in pick
        const uint64_t word =
            __builtin_amdgcn_ballot_w64(a0 + lane < s.nq && over[a0 + lane] != 0);
        const int m = __popcll(word);
        if (m == 0) continue;
        __syncthreads();
        if (tid < 64 && (word >> tid & 1)) pick[__popcll(word & ((1ull << tid) - 1))] = a0 + tid;
        __syncthreads();
        const int slots = m > 1 ? 1 << (32 - __clz(m - 1)) : 1;  // a power of two >= m
        const int slot = tid & (slots - 1);
        if (slot < m) {
          const double q = ((double)pick[slot] + 0.5) * dq;
          const double ex = exp(-2.0 * q * s.d);
          const double kq = q * q * q * ex;
          const double qd = s.dispersion ? q * s.d : 1.0;
          const double W = s.omega_l * s.omega_l + s.v_l * s.v_l * q * q, Al = s.a_l * W;
          double P[kRestNodes], S[kRestNodes];
#pragma unroll
          for (int j = 0; j < kRestNodes; j++) {
            // P = Omega^2 (q d): rounded twice only (next to a resonance P - w^2
            // magnifies its rounding by w / gamma_s)
            P[j] = om2[j] * qd;
            S[j] = 0.0;
          }
          auto sum = [&](int first, int step) {
            for (int b = first; b < nb; b += step) {
              const RestEntry e = tab[b];
              const double dl = W - e.w2;
              const double inv = Al / (dl * dl + e.glw * e.glw);
              const double Il = inv * e.glw, vI = e.v * Il;
              if constexpr (SCREEN) {
                const OmegaTerm t{1.0 - ex * (inv * dl), -ex * Il, e.w2, e.gw, vI};
#pragma unroll
                for (int j = 0; j < kRestNodes; j++) S[j] = omega_sum(t, P[j], S[j]);
              } else {
                const double t = e.gw * e.gw;
#pragma unroll
                for (int j = 0; j < kRestNodes; j++) {
                  const double dd = P[j] - e.w2;
                  S[j] = __builtin_fma(vI, recip_nr(dd * dd + t), S[j]);
                }
              }
            }
          };
          if (slots == 64)  // a wave's omegas, counted in scalar registers
            sum(uniform(wv), 4);
          else
            sum(tid / slots, kQuadThreads / slots);
#pragma unroll
          for (int j = 0; j < kRestNodes; j++) acc[j] += kq * P[j] * S[j];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kRestNodes; j++) {
      const double v = wave_sum(acc[j]);
      if (lane == 0) red[j][wv] = v;
    }
    __syncthreads();
    if (tid < kRestNodes && k0 + tid <= n) {
      double t = 0;
      for (int w = 0; w < kQuadThreads / 64; w++) t += red[tid][w];
      raw[k0 + tid] += quad_scale(s) * t;
    }
    __syncthreads();
  }
}

// Every q point node by node, where the one table is missing: the sums of
// k_friction_raw by a bounded number of blocks, the omega table built once per
// block where it fits.  256 x 1024 points, Omega up to 2 omega0: 129,000 nodes
// 10.8 ms (in k_quad_eval, one node per lane, 22.4; k_friction_raw 10.8), 2580
// nodes 0.41 ms (0.97; 0.37).
__global__ void __launch_bounds__(kQuadThreads) k_quad_all(SpecArgs s,
                                                           const double* __restrict__ omega,
                                                           int64_t n,
                                                           const TabInfo* __restrict__ info,
                                                           double* __restrict__ raw) {
  __shared__ OmegaEntry tab[kQuadTile];
  __shared__ double red[kQuadNodes][kQuadThreads / 64];
  if (info[0].np <= kTabCap) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const double dq = s.q_max / s.nq;
  bool built = false;
  for (int64_t k0 = (int64_t)blockIdx.x * kQuadNodes; k0 <= n;
       k0 += (int64_t)gridDim.x * kQuadNodes) {
    double om2[kQuadNodes], acc[kQuadNodes];
#pragma unroll
    for (int j = 0; j < kQuadNodes; j++) {
      const int64_t k = k0 + j;
      const double o = k < n ? omega[k] : s.omega0;  // k >= n: reference (k == n) or padding
      om2[j] = o * o;
      acc[j] = 0.0;
    }
    for (int b0 = 0; b0 < s.nw; b0 += kQuadTile) {
      const int nb = min(kQuadTile, s.nw - b0);
      if (!built) {
        __syncthreads();
        for (int b = tid; b < nb; b += kQuadThreads) {
          const OmegaTerm t = omega_term(s, 0, b0 + b);
          tab[b] = OmegaEntry{t.br, t.bi * t.bi, t.v, 0.0};
        }
        __syncthreads();
        built = s.nw <= kQuadTile;
      }
      for (int a = tid; a < s.nq; a += kQuadThreads) {
        const double q = ((double)a + 0.5) * dq;
        const double kq = q * q * q * exp(-2.0 * q * s.d);
        const double qd = s.dispersion ? q * s.d : 1.0;
        double P[kQuadNodes], S[kQuadNodes];
#pragma unroll
        for (int j = 0; j < kQuadNodes; j++) {
          P[j] = om2[j] * qd;
          S[j] = 0.0;
        }
        for (int b = 0; b < nb; b++) {
          const OmegaEntry e = tab[b];  // same b for every lane: LDS broadcast
#pragma unroll
          for (int j = 0; j < kQuadNodes; j++) {
            const double dd = P[j] - e.s;
            S[j] = __builtin_fma(e.v, recip_nr(dd * dd + e.t), S[j]);
          }
        }
#pragma unroll
        for (int j = 0; j < kQuadNodes; j++) acc[j] += kq * P[j] * S[j];
      }
    }
#pragma unroll
    for (int j = 0; j < kQuadNodes; j++) {
      const double v = wave_sum(acc[j]);
      if (lane == 0) red[j][wv] = v;
    }
    __syncthreads();
    if (tid < kQuadNodes && k0 + tid <= n) {
      double t = 0;
      for (int w = 0; w < kQuadThreads / 64; w++) t += red[tid][w];
      raw[k0 + tid] = quad_scale(s) * t;
    }
    __syncthreads();
  }
}

__global__ void k_friction_lat(const double* __restrict__ raw, int64_t n, double target,
                               double* __restrict__ lambda) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) lambda[k] = target * raw[k] / raw[n];
}

// ------------------------------------------------------------ launchers
// Tables pay from a number of nodes on: building one costs at most 256 x 20
// points, the node-by-node sum n points per q.  The bounds also see to it that
// one table (or one group of them) fits the scratch of every caller, so that
// the route, and with it the result's bits, depends on n and the spectra
// alone: a context's scratch, a population buffer, has at least 18 bytes per
// wall node (nine halves), and 2560 x 18 holds a shared table, 18432 x 18 a
// group's.
static bool quad_shared(const SpecArgs& s) { return !s.coupling && s.v_l == 0.0; }
static constexpr int64_t kGroupBytes = kTabGroup * (kTabDoubles * 8 + (int64_t)sizeof(TabInfo));
static constexpr int64_t kRangeBytes = kRangeBlocks * 2 * 8;
static constexpr int64_t kSharedBytes = kTabDoubles * 8 + (int64_t)sizeof(TabInfo);
// whether each q has a table (not shared), in whole words for the tables'
// alignment
static int64_t over_bytes(const SpecArgs& s) { return ((int64_t)s.nq + 7) / 8 * 8; }
static_assert(18 * kQuadSharedNodes >= kRangeBytes + kSharedBytes, "scratch");
static_assert(18 * kQuadTableNodes >= kRangeBytes + kGroupBytes + 2560, "scratch");
static constexpr int kMinRows = 4;

hipError_t launch_friction(const SpecArgs& s, const double* omega, int64_t n, double* raw,
                           double* lambda, void* scratch, int64_t scratch_bytes, hipStream_t st) {
  const bool shared = quad_shared(s);
  const int64_t mask = shared ? 0 : over_bytes(s);
  // (above 2560 q points their bytes may need some more nodes: 4096 from 18,503)
  if (n >= (shared ? kQuadSharedNodes : kQuadTableNodes) &&
      std::min(18 * n, scratch_bytes) >=
          kRangeBytes + mask + (shared ? kSharedBytes : kGroupBytes)) {
    char* p = static_cast<char*>(scratch);
    double* range = reinterpret_cast<double*>(p);
    p += kRangeBytes;
    uint8_t* over = reinterpret_cast<uint8_t*>(p);
    p += mask;
    const int64_t left = scratch_bytes - kRangeBytes - mask - (shared ? kSharedBytes : 0);
    const int64_t row = 8 * (n + 1), each = shared ? 0 : kGroupBytes;
    const int total = (s.nq + kTabGroup - 1) / kTabGroup;
    // rows (more blocks in flight) where at least kMinRows of them fit
    int fit = (int)std::min<int64_t>(std::min(total, 4096), left / (row + each));
    const bool rows = fit >= std::min(total, kMinRows);
    if (!rows) fit = shared ? total : (int)std::min<int64_t>(std::min(total, 4096), left / each);
    if (left < 0 || fit < 1) return hipErrorInvalidValue;
    const int ntab = shared ? 1 : fit * kTabGroup;
    TabInfo* info = reinterpret_cast<TabInfo*>(p);
    double* tab = reinterpret_cast<double*>(p + ntab * sizeof(TabInfo));
    double* part = rows ? tab + ntab * kTabDoubles : nullptr;
    const unsigned nblk = (unsigned)((n + 1 + kQuadThreads - 1) / kQuadThreads);
    constexpr unsigned kBuildX = (kTabCap + kBuildPanels - 1) / kBuildPanels;
    hipLaunchKernelGGL(k_quad_range, dim3(kRangeBlocks), dim3(kQuadThreads), 0, st, omega, n,
                       range);
    for (int end = total; end > 0; end -= fit) {
      const int g = std::min(fit, end), g0 = end - g;
      const int tables = shared ? 1 : std::min(g * kTabGroup, s.nq - g0 * kTabGroup);
      if (!shared || end == total) {
        hipLaunchKernelGGL(k_quad_plan, dim3((unsigned)tables), dim3(kQuadThreads), 0, st, s,
                           shared ? 1 : 0, g0 * kTabGroup, range, info, over);
        hipLaunchKernelGGL(k_quad_build, dim3(kBuildX, (unsigned)tables), dim3(kQuadThreads), 0,
                           st, s, shared ? 1 : 0, g0 * kTabGroup, info, tab);
      }
      // a shared table is loaded once per block: several groups each, as long
      // as eight blocks per CU remain (129,024 nodes: 152 -> 133 us)
      const int per =
          !rows ? g : (shared ? (int)std::clamp<int64_t>((int64_t)nblk * g / 2048, 1, g) : 1);
      hipLaunchKernelGGL(k_quad_eval, dim3(nblk, (unsigned)((g + per - 1) / per)),
                         dim3(kQuadThreads), 0, st, s, shared ? 1 : 0, g0, g, per,
                         omega, n, info, tab, part, raw);
      if (rows)
        hipLaunchKernelGGL(k_quad_sum, dim3(nblk), dim3(kQuadThreads), 0, st, s, shared ? 1 : 0,
                           end == total ? 1 : 0, g0 == 0 ? 1 : 0, g, info, part, n, raw);
    }
    // What has no table, node by node.  Some thousand blocks: with nothing to do
    // (the usual case) they are gone in 2 us, and as few as are resident were 9 %
    // slower than blocks that start as others end.
    auto rest_blocks = [n](int nodes) {
      return dim3((unsigned)std::min<int64_t>((n + nodes) / nodes, 4096));
    };
    if (shared)
      hipLaunchKernelGGL(k_quad_all, rest_blocks(kQuadNodes), dim3(kQuadThreads), 0, st, s, omega,
                         n, info, raw);
    else if (s.coupling)
      hipLaunchKernelGGL(k_quad_rest<true>, rest_blocks(kRestNodes), dim3(kQuadThreads), 0, st, s,
                         omega, n, over, raw);
    else
      hipLaunchKernelGGL(k_quad_rest<false>, rest_blocks(kRestNodes), dim3(kQuadThreads), 0, st, s,
                         omega, n, over, raw);
  } else {
    const unsigned blocks = (unsigned)((n + 1 + kQuadNodes - 1) / kQuadNodes);
    if (s.coupling)
      hipLaunchKernelGGL(k_friction_full<true>, dim3(blocks), dim3(kQuadThreads), 0, st, s, omega,
                         n, raw);
    else if (s.v_l != 0.0)
      hipLaunchKernelGGL(k_friction_full<false>, dim3(blocks), dim3(kQuadThreads), 0, st, s, omega,
                         n, raw);
    else
      hipLaunchKernelGGL(k_friction_raw, dim3(blocks), dim3(kQuadThreads), 0, st, s, omega, n, raw);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (n > 0)
    hipLaunchKernelGGL(k_friction_lat, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, raw, n,
                       s.lambda_target, lambda);
  return hipGetLastError();
}

}  // namespace lbm
