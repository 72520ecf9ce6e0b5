// Arguments and launchers of the block form of the adjoint cycle on small meshes (internal). Tiles and
// block counts are those of block_cycle.h.
#pragma once

#include <hip/hip_runtime.h>

namespace mr {

// Uniform offset of a stored lambda: mu = (sum of part[0 .. count)) * scale.
struct AdjMu {
  const double* part;
  int count;
  double scale;
};

struct AdjDownArgs {
  const double* lam;       // lambda in, offset mu (null: zero start)
  const double* rhs;
  const double* coef;      // 6 fields of n^3 (adjoint.hip)
  int n;
  double h2;
  AdjMu mu;
  double* lam_out;
  double* rhs_c;           // 8-son mean of the residual
  double *part_s, *part_r2;   // per block: sum of lambda, sum of the residual's squares
};

struct AdjUpArgs {
  const double* lam;       // offset mu
  const double* rhs;
  const double* coef;
  const double* lam_c;     // coarse correction, offset mu_c
  int n;
  double h2;
  AdjMu mu, mu_c;
  double* lam_out;
  double* part_s;
};

struct AdjTailArgs {
  const double* rhs;       // level of n^3 cells (8, 12, or 10 as the coarsest)
  const double* coef;
  const double* coef_c;    // coarsest level below (unused for 10)
  int n;
  int npre, npost, ncoarse;
  double h2;
  double* lam_out;         // mean-free
};

hipError_t launch_adj_down(const AdjDownArgs& a, hipStream_t s);
hipError_t launch_adj_up(const AdjUpArgs& a, hipStream_t s);
hipError_t launch_adj_tail(const AdjTailArgs& a, hipStream_t s);

}  // namespace mr
