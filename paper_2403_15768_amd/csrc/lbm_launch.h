// lbm_launch.h -- host-side launchers of the kernels in lbm_kernels.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.h"

namespace lbm {

// Spectral parameters as the quadrature kernel takes them (mirrors
// lbm_spectral of the public header).
struct SpecArgs {
  double T, omega0, gamma_s, omega_l, gamma_l, a_l, d;
  int nq, nw;
  double q_max, w_max;
  double lambda_target;
  int dispersion;
  int coupling;  // 1: screening denominator
  double v_l;    // liquid mode dispersion
};


// q: 9 or 19; prec: 0 F64, 1 F32, 2 F16S
hipError_t launch_step(int q, int prec, const void* src, void* dst, const StepArgs& a, bool bouz,
                       hipStream_t st);  // a.ue: electron-sheet walls; a.cellw: masked walls
// one step that also leaves the per-block FP64 (j_x, rho - rho0) partials of
// the populations its collision sees in a.partials (k_moments' blocks and
// order); planar or tube walls without noise, sheets, mask or open ends
hipError_t launch_step_checked(int q, int prec, const void* src, void* dst, const StepArgs& a,
                               bool bouz, hipStream_t st);
// two steps per launch of a small D3Q19 channel (planar or tube walls without
// noise, sheets, mask or open ends, populations of less than 4 GiB): boxes of
// whole x-lines, one per tile; cells (1 or 2) per lane
struct BoxTile {
  int32_t y0, y1, z0, z1;
};
struct BoxArgs {
  int blocks, lanes, cells;
  const BoxTile* tiles;
  const ColInfo* cols;  // per box column
};
hipError_t launch_step_box(int prec, const void* src, void* dst, const StepArgs& a,
                           const BoxArgs& ba, bool bouz, hipStream_t st);
const void* box_kernel_ptr(int prec, bool bouz, int cells);  // (src, dst, StepArgs, BoxArgs)
// two steps per launch of a large D3Q19 channel in double (planar walls, no
// noise, sheets, mask or open ends, populations of less than 4 GiB): tiles of
// tx cells along x (whole x-lines where hx = 0, else with a halo lane on either
// side) times one of `tiles` (its rows and a row on either side fit the lanes)
struct PairArgs {
  int ntiles, xtiles;  // all tiles; tiles along x (they vary fastest)
  int tx, hx;
  const BoxTile* tiles;
  const ColInfo* cols;  // per box column
};
hipError_t launch_step_pair(const void* src, void* dst, const StepArgs& a, const PairArgs& pa,
                            hipStream_t st);
const void* pair_kernel_ptr();  // (src, dst, StepArgs, PairArgs)
int pair_lanes();
// k steps per launch of a D2Q9 slab without noise, sheets or open ends: tiles of tx x ty cells, in LDS
// with k cells on every side (rx = tx + 2 k), or of whole x-lines (rx = tx =
// nx); cells (1 or 2) per lane
struct RunArgs {
  int blocks, lanes;
  int xtiles, tx, ty, rx, k, whole, cells;
  const ColInfo* cols;
};
int run_lanes();  // most lanes of a workgroup
hipError_t launch_step_run(int prec, const void* src, void* dst, const StepArgs& a,
                           const RunArgs& ra, hipStream_t st);
const void* run_kernel_ptr(int prec, int cells);  // (src, dst, StepArgs, RunArgs)
const void* step_kernel_ptr(int q, int prec, bool bouz, int th_mode, bool elec,
                            bool masked, bool open, bool nt);
// one electron step from the water state g (step n): e_src -> e_dst, u_e of
// step n -> ue; the water step of step n then reads ue
hipError_t launch_electron_step(int q, int prec, const void* g, const double* e_src,
                                double* e_dst, double* ue, const ElecArgs& ea, hipStream_t st);
const void* electron_kernel_ptr(int q, int prec);
// both in one launch (slab and duct lines, one workgroup per x-line: a.segs = 1)
hipError_t launch_step_lines(int q, int prec, const void* src, void* dst, const StepArgs& a,
                             const double* e_src, double* e_dst, double* ue, const ElecArgs& ea,
                             hipStream_t st);
// (src, dst, StepArgs, e_src, e_dst, ue, ElecArgs)
const void* lines_kernel_ptr(int q, int prec, int th_mode);
// open x ends: the records of the ghosts beside the first and the last node of
// every column of src ([side][column][kEndSlots] doubles, see end_shifts),
// before the step that reads src
hipError_t launch_open_moments(int q, int prec, const void* src, const StepArgs& a, double* bmom,
                               hipStream_t st);
const void* open_moments_kernel_ptr(int q, int prec);  // (src, StepArgs, bmom)
hipError_t launch_moments(int q, int prec, const void* src, const StepArgs& a, bool bouz,
                          int which, double* field, double* partials, hipStream_t st);
// out[0..4]: sum j_x, sum (rho - rho0), then flux (sum j_x / nx), mass
// (mass0 + sum (rho - rho0)) and the mass deviation; out_host (pinned host
// memory, device pointer) receives the same if not null
hipError_t launch_reduce_final(const double* partials, int64_t nblocks, double* out, int nx,
                               double mass0, hipStream_t st, double* out_host = nullptr);
// the friction quadrature; scratch (device) holds the tables of the piecewise
// sums, which take over from the node-by-node sums at kQuadSharedNodes nodes
// (spectra whose omega sum does not depend on q) or kQuadTableNodes (the
// others).  It needs 1 KiB and one table of 40 KiB, or a group of eight and a
// byte per q point: less than 18 bytes per node from there on, which a
// context's population buffer always has (up to 2560 q points; with more, from
// the node count that gives as much).  The result does not depend on its size.
constexpr int64_t kQuadSharedNodes = 2560, kQuadTableNodes = 18432;
hipError_t launch_friction(const SpecArgs& s, const double* omega, int64_t n, double* raw,
                           double* lambda, void* scratch, int64_t scratch_bytes, hipStream_t st);
hipError_t launch_set_step(int64_t* d, int64_t v, hipStream_t st);
const void* add_step_kernel_ptr();  // k_add_step(int64_t* d, int64_t v)
// storage-precision change (0 F64, 1 F32, 2 F16S) of `rows` x-lines of nx
// populations, nxp_in / nxp_out elements apart
hipError_t launch_convert(int pin, const void* in, int nxp_in, int pout, void* out, int nxp_out,
                          int64_t rows, int nx, hipStream_t st);
// batches
const void* batch_step_kernel_ptr(int q, int prec, bool bouz, int th, bool open,
                                  bool elec);  // th: noise form; open: open x ends
// k_batch_electrons: grid (blocks of 256 line nodes of the largest member,
// members), arguments (md, EGroup, bstep, step_off)
const void* batch_electron_kernel_ptr(int q, int prec);
// k_batch_step(const MemberDesc*, const WorkItem*, const int32_t* cols, int64_t first,
//              int64_t nwall, int64_t last, const int64_t* bstep, int64_t step_off, int wpb)
// per-item partials of the flux and mass of items [first, first + count)
hipError_t launch_batch_moments(int q, int prec, const MemberDesc* md, const WorkItem* items,
                                const int32_t* cols, int64_t first, int64_t count,
                                const int64_t* bstep, double* partials, bool bouz,
                                hipStream_t st);
// per member slot m < nslots: out[2m..2m+1] = sum of the partials of the
// items order[mstart[m] .. mstart[m] + mcount[m])
hipError_t launch_batch_reduce(const double* partials, const int32_t* order, const int64_t* mstart,
                               const int64_t* mcount, int nslots, double* out, hipStream_t st);
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t st);
hipError_t launch_set_r(int prec, const double* lambda, int64_t n, void* r, int* bad,
                        hipStream_t st);

}  // namespace lbm
