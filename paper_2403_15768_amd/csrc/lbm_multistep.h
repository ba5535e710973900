// lbm_multistep.h -- several time steps per launch, in LDS (part of
// lbm_kernels.hip).
//
//  k_step_run       many steps of a tile of a D2Q9 slab
//  k_step_box       two steps of a box of a small D3Q19 channel
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {

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

// ------------------------------------------------------------ D3Q19: two steps
// A channel of up to some 250,000 cells fits the 256 CUs' LDS once; its step
// is bound by the latency of a launch (1.7 us), of its loads, of the update's
// dependent operations and of its stores, not by any rate.  Here a workgroup
// owns a box of whole x-lines and takes two steps of it per launch: the first
// one from memory, on the box and the columns next to it (cut off at walls; a
// slab's z is periodic), into LDS, the second from there to memory.  The
// arithmetic and the random bits are a single step's, so the result is the
// same bit for bit.
//
// Measured per step: duct 32 x 128 x 64 float 11.2 -> 9.4 us, half 13.0 ->
// 7.3; 16 x 64 x 64 double 9.9 -> 5.0, float 8.0 -> 5.0; 32 x 32 x 32 double
// 5.8 -> 4.7, float 6.3 -> 4.8; tube R = 8 of 16 cells double 6.1 -> 4.8.  Boxes
// cut along x as well (rows of 34 lanes) gained nothing, and four steps per
// launch spilled registers (6.8 us for that tube).
constexpr int kBoxLanes = 1024;

template <typename S, typename M, bool BOUZ, int CELLS>
__global__ void __launch_bounds__(kBoxLanes) k_step_box(const S* __restrict__ src,
                                                        S* __restrict__ dst, StepArgs a,
                                                        BoxArgs ba) {
  using L = D3Q19;
  constexpr int N = CELLS * kBoxLanes;
  __shared__ S lds[L::Q * N];
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const BoxTile tile = ba.tiles[blockIdx.x];
  const int yb = max(tile.y0 - 1, 0), ry = min(tile.y1 + 1, ny) - yb;
  const int zb = a.slab ? tile.z0 - 1 : max(tile.z0 - 1, 0);
  const int rz = (a.slab ? tile.z1 + 1 : min(tile.z1 + 1, nz)) - zb;
  const int n = nx * ry * rz, plane = nx * ry;
  const int nt = (int)blockDim.x, tid = (int)threadIdx.x;
  const int64_t step = (a.dstep ? uniform64(*gbl(a.dstep)) : 0) + a.step_off;
  const LBM_GLOBAL S* g = gbl(src);
  const unsigned sI = (unsigned)a.sI, sC = (unsigned)a.sC, sZ = (unsigned)ny * sC;
  const LBM_GLOBAL M* rwall = gbl(static_cast<const M*>(a.rwall));
  const LBM_GLOBAL M* bz = BOUZ ? gbl(static_cast<const M*>(a.bz)) : nullptr;

  // the lane's cells: x, column, wall column and links; whether there is one,
  // and whether it is inside the box
  int x[CELLS], col[CELLS], wc[CELLS];
  bool on[CELLS], in[CELLS];
  uint32_t mask[CELLS];
#pragma unroll
  for (int c = 0; c < CELLS; c++) {
    const int e = tid + c * nt;
    const int lz = e / plane, r2 = e - lz * plane, ly = r2 / nx;
    const int y = yb + ly;
    int z = zb + lz;
    in[c] = y >= tile.y0 && y < tile.y1 && z >= tile.z0 && z < tile.z1;
    z = z < 0 ? z + nz : (z >= nz ? z - nz : z);
    x[c] = r2 - ly * nx;
    col[c] = z * ny + y;
    wc[c] = 0;
    mask[c] = 0u;
    if (e < n) {
      const LBM_GLOBAL ColInfo* ci = gbl(ba.cols) + col[c];
      mask[c] = ci->mask;
      wc[c] = ci->wallcol;
    }
    on[c] = e < n && !(mask[c] & kSolidColumn);
  }

  // the first step, from memory
#pragma unroll
  for (int c = 0; c < CELLS; c++) {
    if (!on[c]) continue;
    const unsigned o0 = (unsigned)col[c] * sC + (unsigned)x[c];
    const unsigned om = x[c] == 0 ? o0 + (unsigned)(nx - 1) : o0 - 1u;
    const unsigned op = x[c] == nx - 1 ? o0 - (unsigned)(nx - 1) : o0 + 1u;
    M df[L::Q];
    if (__builtin_amdgcn_ballot_w64(mask[c] != 0u) == 0) {
      S v[L::Q];
#pragma unroll
      for (int i = 0; i < L::Q; i++)
        v[i] = *at(sbase(g + a.nboff[i]), L::cx[i] > 0 ? om : (L::cx[i] < 0 ? op : o0));
#pragma unroll
      for (int i = 0; i < L::Q; i++) df[i] = dec<S, M>(v[i]);
    } else {
      const int z = col[c] / ny, y = col[c] - z * ny;
      const bool node = (mask[c] & kLinkBits) != 0u;
      const M r = node ? rwall[(int64_t)wc[c] * nx + x[c]] : M(0);
      const LBM_GLOBAL M* cw = BOUZ ? bz + (int64_t)(node ? wc[c] : 0) * L::Q * 2 : nullptr;
      S v[L::Q], b[L::Q];
#pragma unroll
      for (int i = 0; i < L::Q; i++) {
        const bool wall = i != 0 && (mask[c] & (1u << i));
        unsigned from = (L::cx[i] > 0 ? om : (L::cx[i] < 0 ? op : o0)) + (unsigned)a.nboff[i];
        if (L::cz[i] != 0 && (mask[c] & kWrapColumn)) {
          if (z - L::cz[i] < 0) from += (unsigned)nz * sZ;
          if (z - L::cz[i] >= nz) from -= (unsigned)nz * sZ;
        }
        v[i] = *at(g, wall ? o0 + L::row[L::sig[i]] * sI : from);
        if (wall) b[i] = *at(g, o0 + L::row[L::opp[i]] * sI);
      }
#pragma unroll
      for (int i = 0; i < L::Q; i++) {
        const M gs = dec<S, M>(v[i]);
        df[i] = gs;
        if (i == 0 || !(mask[c] & (1u << i))) continue;
        M cb = M(0), cc = M(0), behind = M(0), own = M(0);
        if (BOUZ) {
          cb = cw[2 * i];
          cc = cw[2 * i + 1];
          if (cb != M(0))
            behind = dec<S, M>(*at(g, (L::cx[i] > 0 ? op : (L::cx[i] < 0 ? om : o0)) +
                                          (unsigned)(L::cy[i] * (int)sC + L::cz[i] * (int)sZ) +
                                          L::row[L::opp[i]] * sI));
          if (cc != M(0)) own = dec<S, M>(*at(g, o0 + L::row[i] * sI));
        }
        df[i] = wall_value<L, S, M, BOUZ>(i, a, gs, dec<S, M>(b[i]), r, cb, cc, behind, own, y);
      }
    }
    S* const o = lds + tid + c * nt;
    collide<L, M, S>(df, a, (uint32_t)col[c] * (uint32_t)nx + (uint32_t)x[c], step,
                     (const M*)nullptr, (M*)nullptr, [&](int i, S e) { o[i * N] = e; });
  }
  __syncthreads();

  // the second, from LDS
#pragma unroll
  for (int c = 0; c < CELLS; c++) {
    if (!on[c] || !in[c]) continue;
    const int l0 = tid + c * nt;
    const int lm = x[c] == 0 ? l0 + nx - 1 : l0 - 1;
    const int lp = x[c] == nx - 1 ? l0 - (nx - 1) : l0 + 1;
    M df[L::Q];
    auto place = [&](int cx, int cy, int cz) {
      return (cx > 0 ? lp : (cx < 0 ? lm : l0)) + cy * nx + cz * plane;
    };
    if (__builtin_amdgcn_ballot_w64((mask[c] & kLinkBits) != 0u) == 0) {
      S v[L::Q];
#pragma unroll
      for (int i = 0; i < L::Q; i++)
        v[i] = lds[i * N + place(-L::cx[i], -L::cy[i], -L::cz[i])];
#pragma unroll
      for (int i = 0; i < L::Q; i++) df[i] = dec<S, M>(v[i]);
    } else {
      const bool node = (mask[c] & kLinkBits) != 0u;
      const M r = node ? rwall[(int64_t)wc[c] * nx + x[c]] : M(0);
      const LBM_GLOBAL M* cw = BOUZ ? bz + (int64_t)(node ? wc[c] : 0) * L::Q * 2 : nullptr;
      const int y = col[c] % ny;
#pragma unroll
      for (int i = 0; i < L::Q; i++) {
        const bool wall = i != 0 && (mask[c] & (1u << i));
        const int from = i * N + place(-L::cx[i], -L::cy[i], -L::cz[i]);
        const M gs = dec<S, M>(lds[wall ? L::sig[i] * N + l0 : from]);
        df[i] = gs;
        if (i == 0 || !wall) continue;
        M cb = M(0), cc = M(0), behind = M(0), own = M(0);
        if (BOUZ) {
          cb = cw[2 * i];
          cc = cw[2 * i + 1];
          if (cb != M(0))
            behind = dec<S, M>(lds[L::opp[i] * N + place(L::cx[i], L::cy[i], L::cz[i])]);
          if (cc != M(0)) own = dec<S, M>(lds[i * N + l0]);
        }
        df[i] = wall_value<L, S, M, BOUZ>(i, a, gs, dec<S, M>(lds[L::opp[i] * N + l0]), r, cb,
                                           cc, behind, own, y);
      }
    }
    const uint32_t cell = (uint32_t)col[c] * (uint32_t)nx + (uint32_t)x[c];
    collide_store<L, M, S>(df, a, gbl(dst), (unsigned)col[c] * sC + (unsigned)x[c], cell, step + 1);
  }
}

// cells = 2: float and half storage (a box of doubles fills LDS with one)
const void* box_kernel_ptr(int prec, bool bouz, int cells) {
#define BK(S, M, C)                                                     \
  (bouz ? reinterpret_cast<const void*>(&k_step_box<S, M, true, C>)     \
        : reinterpret_cast<const void*>(&k_step_box<S, M, false, C>))
  if (prec == 0) return BK(double, double, 1);
  if (prec == 1) return cells == 1 ? BK(float, double, 1) : BK(float, double, 2);
  return cells == 1 ? BK(_Float16, float, 1) : BK(_Float16, float, 2);
#undef BK
}

hipError_t launch_step_box(int prec, const void* src, void* dst, const StepArgs& a,
                           const BoxArgs& ba, bool bouz, hipStream_t st) {
  StepArgs args = a;
  BoxArgs bargs = ba;
  void* kargs[4] = {(void*)&src, (void*)&dst, (void*)&args, (void*)&bargs};
  return hipLaunchKernel(box_kernel_ptr(prec, bouz, ba.cells), dim3((unsigned)ba.blocks),
                         dim3((unsigned)ba.lanes), kargs, 0, st);
}

}  // namespace lbm
