// Arguments and launchers of the block form of the FAS cycle on small meshes (internal).
#pragma once

#include <hip/hip_runtime.h>

namespace mr {

constexpr int kBlkMaxN = 80;        // largest level of the block form
constexpr int kBlkMaxBlocks = 512;  // blocks (partial sums) of a launch

// Shift of a launch: C = c_scale * (sum of c_part[0 .. c_count)).
struct BlkDownArgs {
  const double* theta;     // iterate in (colour-split, as every field)
  const double* delta;
  const double* rd;        // restricted defect (null on the finest level: no right-hand side)
  int n;
  double h2, ih2;
  const double* c_part;
  int c_count;
  double c_scale;
  double* theta_out;       // smoothed iterate
  double* f_out;           // FAS right-hand side (with rd)
  double* theta_c;         // 8-son means on the coarse level: theta, defect
  double* rd_c;
  double *part_c, *part_d, *part_d2;   // per block: Sigma + f of the last sweep, defect, defect^2
  double* c_out;           // receives C (may be null)
};

struct BlkUpArgs {
  const double* theta;     // pre-smoothed iterate
  const double* delta;
  const double* f;         // null on the finest level
  const double* theta_c;   // coarse solution and its start
  const double* that_c;
  int n;
  double h2, ih2;
  const double* c_part;
  int c_count;
  double c_scale;
  double* theta_out;
  double* part_c;
};

struct BlkTailArgs {
  const double* that;      // restricted theta of the level of n^3 cells (n <= 12)
  const double* delta;
  const double* rd;
  const double* delta_c;   // delta of the coarsest level below (unused with coarsest)
  int n;
  int coarsest;            // the level itself is the coarsest one
  int npre, npost, ncoarse;
  double h2, ih2;
  const double* c_part;
  int c_count;
  double c_scale;
  double* theta_out;
};

struct BlkTile {
  int ti, tj, tk;
};
BlkTile blk_tile(int n);   // tile of a level of n^3 cells (ti == 0: none)
bool blk_level_supported(int n);
int blk_blocks(int n);
hipError_t launch_blk_down(const BlkDownArgs& a, hipStream_t s);
hipError_t launch_blk_up(const BlkUpArgs& a, hipStream_t s);
hipError_t launch_blk_tail(const BlkTailArgs& a, hipStream_t s);

}  // namespace mr
