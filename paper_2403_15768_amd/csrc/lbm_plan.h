// lbm_plan.h -- the tiles of the two-step kernel of large channels in double,
// and whether it pays (host only, plain values).
#pragma once

#include <algorithm>
#include <cstdint>

namespace lbm {

// Tiles of tx cells along x (hx = 0: whole x-lines; hx = 1: with a halo lane on
// either side) times ty rows times lz planes; tx = 0: single steps are faster.
struct PairPlan {
  int hx = 0, tx = 0, ty = 0, lz = 0;
};

// Times in us by a model fitted to 300 measurements of 220 channels, 1 to 32768
// cells long and of one to 512 rows and planes (6 % rms): channels in double of
// at least 2^18 cells, 256 CUs.  On 110 other channels its choice was slower
// than single steps once (4 %) and missed 4 to 10 % three times.  `far`: the
// share of the state (both buffers, mb in MB) that the 256 MB last-level cache
// no longer keeps.
inline double pair_far(double mb) { return std::min(1.0, std::max(0.0, (mb - 255.0) / 35.0)); }

// One step per launch: by the cells, padding included, and by the columns and
// the waves where the lines are short or fill their waves badly (16 x 128 x 128
// 21 us, 73 x 118 x 33 16.6; 64 x 64 x 64 13.1).
inline double single_step_us(int nx, int nxp, int ny, int nz) {
  const double cols = (double)ny * nz, far = pair_far(cols * nxp * 304e-6);
  const double per_cell = nx <= 128 && nx % 8 ? 0.0487 : 0.0462;
  const double near_line =
      std::max({per_cell * nxp, 1.0 + 0.027 * nxp, 1.95 * ((nx + 63) / 64)});
  const double far_line = std::max(near_line, (nx < 400 ? 0.052 : 0.057) * nxp);
  return 1.3 + 1e-3 * cols * ((1.0 - far) * near_line + far * far_line);
}

// The pair kernel's two steps: rounds of at most 256 tiles, each a pass per
// plane and two for the halo's (less where that plane lies beyond a wall).  A
// pass takes the latency of its chain -- more where every tile holds both y
// walls, less where fewer CUs are busy -- or, once the state comes from memory,
// the time of its cells' traffic.
inline double pair_steps_us(bool slab, int nxp, int ny, int nz, const PairPlan& p, int64_t tiles) {
  const int64_t rounds = (tiles + 255) / 256;
  const double each = (double)tiles / rounds;  // tiles of a round
  const int zt = (nz + p.lz - 1) / p.lz;
  const double passes = rounds * (p.lz + 2 - (slab || zt > 2 ? 0.0 : 0.7 / zt));
  const double one_round =
      (slab ? 2.9 : 3.0) + 1.5 * std::min(1.0, each / 200.0) + (p.hx ? 0.2 : 0.0);
  const double near_pass = (rounds > 1 ? 4.15 : one_round) + (p.ty >= ny ? 0.3 : 0.0);
  const double stored = 1e-3 * std::max(each, 224.0) * p.tx * p.ty * p.lz / (p.lz + 2);
  const double far_pass = std::max(near_pass, (p.hx ? 2.5 : 2.1) + 0.045 * stored);
  const double far = pair_far((double)ny * nz * nxp * 304e-6);
  return 3.0 + passes * ((1.0 - far) * near_pass + far * far_pass);
}

// Whole x-lines (where they are stored back to back: nxp = nx) or 32 cells
// (whole cache lines) with a halo, each with the range of z of the fewest
// passes; none where single steps are not 4 % slower at least.  Measured per
// step, single -> pair: 256 x 128 x 64 107.7 -> 82.2 us, 96 x 128 x 64 36.5 -> 25.7
// (32 cells; whole lines 34.3), 64 x 128 x 64 24.6 -> 19.0 (whole lines; 32 cells
// 20.7), 112 x 100 x 60 31.5 -> 25.0 (whole lines 33.4).  Not taken: slabs of one
// to three planes (1024 x 128 x 2 13.6 -> 17.6), 256 x 32 x 32 (13.3 -> 15.0),
// 300 x 7 x 200 (21.7 -> 26.5).
inline PairPlan choose_pair(bool slab, int nx, int nxp, int ny, int nz, int lanes) {
  PairPlan best;
  double us = 2.0 * 0.96 * single_step_us(nx, nxp, ny, nz);
  for (int hx = nxp <= 128 ? 0 : 1; hx <= 1; hx++) {
    PairPlan p;
    p.hx = hx;
    p.tx = hx ? 32 : nx;
    const int rows = lanes / (p.tx + 2 * hx) - 2;
    if (rows < 1) continue;
    const int64_t xt = (nxp + p.tx - 1) / p.tx, yt = (ny + rows - 1) / rows;
    p.ty = (int)((ny + yt - 1) / yt);
    int64_t fewest = INT64_MAX;
    for (int lz = 1; lz <= nz; lz++) {
      const int64_t passes = (xt * yt * ((nz + lz - 1) / lz) + 255) / 256 * (lz + 2);
      if (passes < fewest) {
        fewest = passes;
        p.lz = lz;
      }
    }
    const double t = pair_steps_us(slab, nxp, ny, nz, p, xt * yt * ((nz + p.lz - 1) / p.lz));
    if (t < (best.tx ? 0.96 * us : us)) {  // (a near tie: whole lines)
      us = t;
      best = p;
    }
  }
  return best;
}

}  // namespace lbm
