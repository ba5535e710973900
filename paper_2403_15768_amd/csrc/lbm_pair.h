// lbm_pair.h -- two time steps per launch of large D3Q19 channels in double
// (part of lbm_kernels.hip).
//
//  k_step_pair      a workgroup owns a tile of (x, y) and a range of z and
//                   marches along z: the first step of plane p on the tile
//                   and its halo, then the second step of plane p - 1 on the
//                   tile, whose pulls read the first step's planes from LDS
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.h"
#include "lbm_launch.h"

namespace lbm {

// One step per launch reads and writes the whole state, and the memory system
// bounds it (the 256 x 128 x 64 duct in double: 637.7 MB in 108 us, as fast as
// a plain copy).  Two steps per launch nearly halve that traffic (counters:
// 698 MB for two); the price is the first step of the tile's halo, computed
// by every tile that needs it, with the same arithmetic, so that the result
// is that of two single steps bit for bit.
//
// Lane = one cell (x, y) of the tile with its halo; the halo along x is left
// out where the tile holds whole x-lines.  LDS holds of each lane's
// first-step populations, by the plane they were computed on: c_z = +1 of
// three planes, c_z = 0 (without the rest population) of two, c_z = -1 of one:
// 36 values a lane, 512 lanes of doubles in 160 KB.  The others that the
// second step needs are the lane's own: the rest population and, for wall
// links, c_z = -1 of the plane before, in registers.  The pulls of the next
// plane are in flight while the second step computes.
//
// Measured per step: 256 x 128 x 64 108.4 -> 82.2 us, 320 x 128 x 64 137.1 ->
// 97.9, 200 x 100 x 60 69.8 -> 57.2, 64 x 128 x 64 24.5 -> 19.2, 40 x 120 x 60
// 15.5 -> 13.8 (lbm_plan.h: the tiles, and the channels that keep single steps).
// What bounds it now is latency with two waves per SIMD (VALU
// busy for a quarter of the time).  Float storage was slower this way (53 ->
// 79 us: its arithmetic is double too, and its rounding adds to it), half
// storage (28 -> 44 us) and interpolated walls (95 -> 107 us) as well.
constexpr int kPairLanes = 512;
constexpr int kPairUp = 5, kPairMid = 8, kPairDown = 5;
constexpr int kPairSlots = 3 * kPairUp + 2 * kPairMid + kPairDown;

// slot of direction i among the directions of its c_z (rest: none)
template <class L>
constexpr int pair_slot(int i) {
  int k = 0;
  for (int j = 1; j < i; j++)
    if (L::cz[j] == L::cz[i]) k++;
  return k;
}

// A barrier that orders LDS only: loads and stores of the state stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__global__ void __launch_bounds__(kPairLanes, 2)
    k_step_pair(const double* __restrict__ src, double* __restrict__ dst, StepArgs a,
                PairArgs pa) {
  using L = D3Q19;
  constexpr int NT = kPairLanes;
  __shared__ double lds[kPairSlots * NT];
  // neighbouring tiles on one XCD (workgroups go round the eight XCDs in
  // turn), so that the halo one reads is in the L2 of the other
  const int per = (pa.ntiles + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || t >= pa.ntiles) return;
  const int tx = t % pa.xtiles;
  const BoxTile tile = pa.tiles[t / pa.xtiles];
  const int tid = threadIdx.x;
  const int rx = pa.tx + 2 * pa.hx;
  const int ly = tid / rx, lx = tid - ly * rx;
  // The lane's place in the tile and its halo, and its cell.  Behind the lane
  // of the halo's cell 0 (xl = nx), padding lanes take cell nx - 1 and store
  // it one place before their own.
  const int xl = tx * pa.tx + lx - pa.hx, y = tile.y0 + ly - 1;
  const int x = xl < 0 || xl > a.nx ? a.nx - 1 : (xl == a.nx ? 0 : xl);
  const int xs = xl > a.nx ? xl - 1 : xl;  // where it is stored
  const bool in1 = ly < tile.y1 - tile.y0 + 2 && y >= 0 && y < a.ny && (xl <= a.nx || xs < a.nxp);
  const bool in2 = ly >= 1 && ly <= tile.y1 - tile.y0 && lx >= pa.hx && xl != a.nx && xs < a.nxp &&
                   (lx < pa.hx + pa.tx || xl > a.nx);
  const unsigned sI = (unsigned)a.sI, sC = (unsigned)a.sC, sZ = (unsigned)a.ny * sC;
  const LBM_GLOBAL double* g = gbl(src);
  const LBM_GLOBAL double* rwall = gbl(static_cast<const double*>(a.rwall));
  const int nz = a.nz;

  const unsigned line = (unsigned)y * sC;
  unsigned o0 = line + (unsigned)x;
  unsigned om = line + (unsigned)(x == 0 ? a.nx - 1 : x - 1);
  unsigned op = line + (unsigned)(x == a.nx - 1 ? 0 : x + 1);
  // this cell's place in LDS, and those at x - 1, x + 1
  const int row = ly * rx;
  int l0 = pa.hx ? row + (xl > a.nx ? x : xl) - tx * pa.tx + 1 : tid;
  int lm = pa.hx ? l0 - 1 : row + (lx == 0 ? a.nx - 1 : lx - 1);
  int lp = pa.hx ? l0 + 1 : row + (lx == a.nx - 1 ? 0 : lx + 1);
  // parts of LDS, as places of slot 0: c_z = +1 of planes p - 2, p - 1, p;
  // c_z = 0 of planes p - 1, p; c_z = -1 of plane p
  int u2 = 0, u1 = kPairUp * NT, u0 = 2 * kPairUp * NT;
  int m1 = 3 * kPairUp * NT, m0 = m1 + kPairMid * NT;
  constexpr int kDown = (3 * kPairUp + 2 * kPairMid) * NT;

  auto wrap = [&](int p) { return a.slab ? (p < 0 ? p + nz : (p >= nz ? p - nz : p)) : p; };
  auto info_of = [&](int p) {  // the lane's column of plane p (none: solid)
    ColInfo ci{-1, kSolidColumn};
    const int pw = wrap(p);
    if (in1 && pw >= 0 && pw < nz) {
      const LBM_GLOBAL ColInfo* c = gbl(pa.cols) + (pw * a.ny + y);
      ci.wallcol = c->wallcol;
      ci.mask = c->mask;
    }
    return ci;
  };
  auto plane_off = [&](int pw, int d) {  // of plane pw + d (periodic)
    int q = pw + d;
    if (q < 0) q += nz;
    if (q >= nz) q -= nz;
    return (unsigned)q * sZ;
  };
  // the pulls of the first step on plane p (a wall link: its partner)
  auto load = [&](int p, const ColInfo& ci, double* v) {
    if (ci.mask & kSolidColumn) return;
    const int pw = wrap(p);
    const bool walls = __builtin_amdgcn_ballot_w64((ci.mask & kLinkBits) != 0u) != 0;
#pragma unroll
    for (int i = 0; i < L::Q; i++) {
      const unsigned u =
          plane_off(pw, -L::cz[i]) + (unsigned)((int)(L::row[i] * sI) - L::cy[i] * (int)sC);
      const unsigned o = L::cx[i] > 0 ? om : (L::cx[i] < 0 ? op : o0);
      if (!walls || i == 0)
        v[i] = *at(g, o + u);
      else if (ci.mask & (1u << i))
        v[i] = *at(g, o0 + (unsigned)pw * sZ + L::row[L::sig[i]] * sI);
      else
        v[i] = *at(g, o + u);
    }
  };

  double dn[kPairDown] = {}, dn_last[kPairDown];  // this lane's c_z = -1 of planes p, p - 1
  double rest = 0.0, rest_last;
  double v[L::Q] = {};
  const int64_t step = (a.dstep ? uniform64(*gbl(a.dstep)) : 0) + a.step_off;
  ColInfo before{-1, kSolidColumn}, info = info_of(tile.z0 - 1);
  load(tile.z0 - 1, info, v);
  for (int p = tile.z0 - 1; p <= tile.z1; p++) {
    // opaque from one plane to the next: the offsets derived from them are
    // formed where they are used, not kept for the whole march
    asm volatile("" : "+v"(o0), "+v"(om), "+v"(op), "+v"(l0), "+v"(lm), "+v"(lp));
    const int pw = wrap(p);
    ColInfo next{-1, kSolidColumn};
    if (p < tile.z1) next = info_of(p + 1);
    const bool on = !(info.mask & kSolidColumn);
    double df[L::Q];
#pragma unroll
    for (int i = 0; i < L::Q; i++) df[i] = v[i];
    if (on && (info.mask & kLinkBits)) {
      const double r = rwall[(int64_t)info.wallcol * a.nx + x];
      double b[L::Q];
#pragma unroll
      for (int i = 1; i < L::Q; i++)
        if (info.mask & (1u << i))
          b[i] = *at(g, o0 + (unsigned)pw * sZ + L::row[L::opp[i]] * sI);
#pragma unroll
      for (int i = 1; i < L::Q; i++)
        if (info.mask & (1u << i))
          df[i] = wall_value<L, double, double, false>(i, a, df[i], b[i], r, 0.0, 0.0, 0.0, 0.0, y);
    }
    lds_barrier();  // the second step of plane p - 2 has read its planes
#pragma unroll
    for (int k = 0; k < kPairDown; k++) dn_last[k] = dn[k];
    rest_last = rest;
    if (on)
      collide<L, double, double>(
          df, a, 0u, step, (const double*)nullptr, (double*)nullptr, [&](int i, double e) {
            if (i == 0) {
              rest = e;
              return;
            }
            lds[(L::cz[i] > 0 ? u0 : (L::cz[i] < 0 ? kDown : m0)) + pair_slot<L>(i) * NT + tid] = e;
            if (L::cz[i] < 0) dn[pair_slot<L>(i)] = e;
          });
    load(p + 1, next, v);  // (a solid column: nothing)
    lds_barrier();
    if (p > tile.z0 && in2 && !(before.mask & kSolidColumn)) {
      const int z = p - 1;  // inside the tile: no wrap
      const uint32_t mask = before.mask;
      double f2[L::Q];
      f2[0] = rest_last;
#pragma unroll
      for (int i = 1; i < L::Q; i++)
        f2[i] = lds[(L::cz[i] > 0 ? u2 : (L::cz[i] < 0 ? kDown : m1)) + pair_slot<L>(i) * NT +
                    (L::cx[i] > 0 ? lm : (L::cx[i] < 0 ? lp : l0)) - L::cy[i] * rx];
      if (mask & kLinkBits) {  // wall links: replace what was read there
        const double r = rwall[(int64_t)before.wallcol * a.nx + x];
        // this lane's own population k of plane z (LDS, or registers for c_z < 0)
        auto own = [&](int k) {
          if (L::cz[k] < 0) return dn_last[pair_slot<L>(k)];
          return lds[(L::cz[k] > 0 ? u1 : m1) + pair_slot<L>(k) * NT + l0];
        };
#pragma unroll
        for (int i = 1; i < L::Q; i++)
          if (mask & (1u << i))
            f2[i] = wall_value<L, double, double, false>(i, a, own(L::sig[i]), own(L::opp[i]), r,
                                                         0.0, 0.0, 0.0, 0.0, y);
      }
      collide_store<L, double, double>(f2, a, gbl(dst), (unsigned)z * sZ + line + (unsigned)xs, 0u,
                                       step + 1);
    }
    before = info;
    info = next;
    const int u = u2;
    u2 = u1;
    u1 = u0;
    u0 = u;
    const int m = m1;
    m1 = m0;
    m0 = m;
  }
}

int pair_lanes() { return kPairLanes; }
const void* pair_kernel_ptr() { return reinterpret_cast<const void*>(&k_step_pair); }

hipError_t launch_step_pair(const void* src, void* dst, const StepArgs& a, const PairArgs& pa,
                            hipStream_t st) {
  StepArgs args = a;
  PairArgs pargs = pa;
  void* kargs[4] = {(void*)&src, (void*)&dst, (void*)&args, (void*)&pargs};
  return hipLaunchKernel(pair_kernel_ptr(), dim3((unsigned)((pa.ntiles + 7) / 8 * 8)),
                         dim3(kPairLanes), kargs, 0, st);
}

}  // namespace lbm
