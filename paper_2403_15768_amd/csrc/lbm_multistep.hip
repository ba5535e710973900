// lbm_multistep.hip -- several time steps per launch, in LDS (D2Q9 slabs).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {

// the mixing weight of a wall node (0 elsewhere)
template <typename M>
__device__ __forceinline__ M wall_r(const StepArgs& a, uint32_t mask, int wallcol, int x) {
  return (mask & kLinkBits) != 0u
             ? gbl(static_cast<const M*>(a.rwall))[(int64_t)wallcol * a.nx + x]
             : M(0);
}

// ------------------------------------------------------------ D2Q9: many steps
// A 2-D channel is a few hundred kilobytes: a step on its own takes as long
// as a launch.  Here a workgroup owns tx x ty cells, loads them with k cells
// on every side (none beyond a wall) into LDS and takes k steps there, the
// outer cells falling out one by one (or, where whole x-lines fit, none of
// them along x: rx = nx).  The arithmetic and the random bits are a single
// step's, so the result is the same bit for bit.  Lanes run along y first, so
// that whole waves fall out.  A step is a chain of LDS reads, the update's
// dependent operations and a barrier: 0.6 us, against 2.6 us for a launch.
// Measured per step, FP64: 64 x 30 cells 2.57 -> 1.23 us, 16 x 8 2.56 ->
// 0.70, 128 x 64 2.68 -> 1.43, 512 x 128 4.60 -> 2.58, 1024 x 128 6.84 -> 3.55;
// FP32 256 x 32 3.01 -> 1.53.
constexpr int kRunLanes = 1024;

// The populations the collision of one cell sees, from one copy of the state
// in LDS, p[direction * N + place] (l0: the cell's place, lm and lp: those at
// x - 1 and x + 1; neighbours along y at place +- 1).  No branches: a lane
// next to a wall reads its own partner population in place of the pull and
// the bounced one beside it (a first version with a branch per link took
// 2.3 us a step against 0.7).
template <class L, typename S, typename M, int N>
__device__ __forceinline__ void gather_run(const S* p, int l0, int lm, int lp, const StepArgs& a,
                                           uint32_t mask, M r, M* df) {
  S v[L::Q], b[L::Q];
#pragma unroll
  for (int i = 0; i < L::Q; i++) {
    const int from = (L::cx[i] > 0 ? lm : (L::cx[i] < 0 ? lp : l0)) - L::cy[i] + i * N;
    const bool wall = L::cy[i] != 0 && (mask & (1u << i));
    v[i] = p[wall ? l0 + L::sig[i] * N : from];
    b[i] = L::cy[i] != 0 ? p[l0 + L::opp[i] * N] : S(0);
  }
#pragma unroll
  for (int i = 0; i < L::Q; i++) {
    const M gs = dec<S, M>(v[i]);
    df[i] = gs;
    if (L::cy[i] == 0) continue;
    const bool wall = mask & (1u << i);
    const M gb = dec<S, M>(b[i]);
    const M mixed = gs + r * (gb - gs);
    df[i] = wall ? mixed : gs;
    if (a.utop != 0.0 && L::cy[i] == -1) {
      const M moving = gb + static_cast<M>(6.0 * L::w[i] * a.rho0 * L::cx[i] * a.utop);
      df[i] = wall ? moving : gs;  // a link with c_y = -1 pulls from the top wall
    }
  }
}

// CELLS cells per lane: one with the steps alternating between two copies in
// LDS (one barrier a step), or two in one copy (two barriers).
template <typename S, typename M, int CELLS>
__global__ void __launch_bounds__(kRunLanes) k_step_run(const S* __restrict__ src,
                                                        S* __restrict__ dst, StepArgs a,
                                                        RunArgs ra) {
  using L = D2Q9;
  constexpr int N = CELLS * kRunLanes;
  constexpr int kCopies = CELLS == 1 ? 2 : 1;
  __shared__ S lds[kCopies * L::Q * N];
  const int nx = a.nx, rx = ra.rx, k = ra.k;
  const int bx = (int)blockIdx.x % ra.xtiles, by = (int)blockIdx.x / ra.xtiles;
  const int x0 = bx * ra.tx, y0 = by * ra.ty;  // first cell of the tile
  const int halo = ra.whole ? 0 : k;
  // rows of the region: yb <= y < yb + ry; a row is lost per step at an end
  // that is no wall
  const int yb = max(y0 - k, 0), ry = min(y0 + ra.ty + k, a.ny) - yb;
  const int lose_lo = yb > 0 ? 1 : 0, lose_hi = yb + ry < a.ny ? 1 : 0;
  const int n = rx * ry;
  const int nt = (int)blockDim.x, tid = (int)threadIdx.x;
  const int64_t step = (a.dstep ? uniform64(*gbl(a.dstep)) : 0) + a.step_off;
  const LBM_GLOBAL S* g = gbl(src) + (int64_t)yb * a.sC;
  for (int e = tid; e < n; e += nt) {
    const int y = e / rx, lx = e - y * rx;
    int x = x0 - halo + lx;
    x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    const LBM_GLOBAL S* c = g + (int64_t)y * a.sC + x;
#pragma unroll
    for (int i = 0; i < L::Q; i++) lds[i * N + lx * ry + y] = c[L::row[i] * a.sI];
  }
  // the lane's cells: place, x and y of the region, number, wall links and r
  int l0[CELLS], lx[CELLS], ly[CELLS];
  uint32_t cell[CELLS], mask[CELLS];
  M r[CELLS];
#pragma unroll
  for (int c = 0; c < CELLS; c++) {
    l0[c] = tid + c * nt;
    lx[c] = l0[c] / ry;
    ly[c] = l0[c] - lx[c] * ry;
    int x = x0 - halo + lx[c];
    x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    cell[c] = (uint32_t)(yb + ly[c]) * (uint32_t)nx + (uint32_t)x;
    mask[c] = 0u;
    r[c] = M(0);
    if (l0[c] < n) {
      const LBM_GLOBAL ColInfo* ci = gbl(ra.cols) + (yb + ly[c]);
      mask[c] = ci->mask & kLinkBits;
      r[c] = wall_r<M>(a, mask[c], ci->wallcol, x);
    } else {
      lx[c] = -1;  // no cell
    }
  }
  __syncthreads();
  S* cur = lds;
  S* nxt = lds + (kCopies - 1) * L::Q * N;
  for (int j = 0; j < k; j++) {
    // lo <= lx < hi, lo_y <= ly < hi_y are updated
    const int lo = ra.whole ? 0 : j + 1, hi = ra.whole ? rx : rx - 1 - j;
    const int lo_y = lose_lo * (j + 1), hi_y = ry - lose_hi * (j + 1);
    M df[CELLS][L::Q];
    bool on[CELLS];
#pragma unroll
    for (int c = 0; c < CELLS; c++) {
      on[c] = lx[c] >= lo && lx[c] < hi && ly[c] >= lo_y && ly[c] < hi_y;
      if (on[c])
        gather_run<L, S, M, N>(cur, l0[c], l0[c] + (lx[c] == 0 ? n - ry : -ry),
                               l0[c] + (lx[c] == rx - 1 ? ry - n : ry), a, mask[c], r[c], df[c]);
    }
    if (kCopies == 1) __syncthreads();
#pragma unroll
    for (int c = 0; c < CELLS; c++)
      if (on[c]) {
        S* const o = nxt + l0[c];
        collide<L, M, S>(df[c], a, cell[c], step + j, (const M*)nullptr, (M*)nullptr,
                         [&](int i, S e) { o[i * N] = e; });
      }
    __syncthreads();
    S* const t = cur;
    cur = nxt;
    nxt = t;
  }
  LBM_GLOBAL S* out = gbl(dst);
  const int ty = min(ra.ty, a.ny - y0);
  // padding behind the last cell (where lines are padded): cell nx - 1's last
  // step again, each with its own random bits, as a single step leaves them
  if (kCopies == 2 && a.nxp > nx && nx - 1 - x0 < ra.tx) {
    const int last = halo + nx - 1 - x0, npad = a.nxp - nx;
    for (int e = tid; e < npad * ty; e += nt) {
      const int q = e / ty, y = y0 + e - q * ty, p0 = last * ry + y - yb;
      const LBM_GLOBAL ColInfo* ci = gbl(ra.cols) + y;
      const uint32_t mk = ci->mask & kLinkBits;
      M df[L::Q];
      gather_run<L, S, M, N>(nxt, p0, p0 - ry, last == rx - 1 ? y - yb : p0 + ry, a, mk,
                             wall_r<M>(a, mk, ci->wallcol, nx - 1), df);
      collide_store<L, M, S>(df, a, out, (unsigned)(y * (int)a.sC + nx + q),
                             (uint32_t)y * (uint32_t)nx + (uint32_t)(nx + q), step + k - 1);
    }
  }
  for (int e = tid; e < ra.tx * ty; e += nt) {
    const int y = e / ra.tx, l = e - y * ra.tx;
    if (x0 + l >= nx) continue;
    LBM_GLOBAL S* o = out + (int64_t)(y0 + y) * a.sC + x0 + l;
#pragma unroll
    for (int i = 0; i < L::Q; i++)
      o[L::row[i] * a.sI] = cur[i * N + (l + halo) * ry + y0 + y - yb];
  }
}

int run_lanes() { return kRunLanes; }
const void* run_kernel_ptr(int prec, int cells) {
#define RK(S, M)                                                     \
  (cells == 1 ? reinterpret_cast<const void*>(&k_step_run<S, M, 1>) \
              : reinterpret_cast<const void*>(&k_step_run<S, M, 2>))
  if (prec == 0) return RK(double, double);
  if (prec == 1) return RK(float, double);
  return RK(_Float16, float);
#undef RK
}

hipError_t launch_step_run(int prec, const void* src, void* dst, const StepArgs& a,
                           const RunArgs& ra, hipStream_t st) {
  StepArgs args = a;
  RunArgs rargs = ra;
  void* kargs[4] = {(void*)&src, (void*)&dst, (void*)&args, (void*)&rargs};
  return hipLaunchKernel(run_kernel_ptr(prec, ra.cells), dim3((unsigned)ra.blocks), dim3((unsigned)ra.lanes),
                         kargs, 0, st);
}

}  // namespace lbm
