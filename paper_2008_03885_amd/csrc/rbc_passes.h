// rbc_passes.h -- the two passes of a red-black coarsening level (rbc_passes.hip): the half
// of a cycle before the coarse correction and the half after it, one launch each.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

namespace mgk {

// A level's stencil on its storage grid: centre, axis +-1, diagonal, axis +-2.
struct RbcOp {
  double c0, a1, d1, a2;
};

// Smallest storage side the passes take (the folds of a rotated level's halo reach five
// points past the boundary).
constexpr int kRbcPassSide = 17;

// One red-black sweep (F points, then C points) of u (null: the zero iterate) into uout,
// then, with fc, the defect restricted onto the next level (zero off its unknowns).
// uc (may be null): the next level's iterate, zeroed.  partials (standard levels, may be
// null): per-block sums of the squared defect of the input u over the interior; *np the
// number of blocks.  uout != u.  done (may be null): the launch does nothing when set.
hipError_t launch_rbc_pre(bool odd, const RbcOp &op, double omega, const double *f, const double *u,
                          double *uout, double *fc, double *uc, int m, double *partials, int *np,
                          const int *done, hipStream_t s);
// uout = one red-black sweep of (uin + the interpolated correction e of the next level).
hipError_t launch_rbc_post(bool odd, const RbcOp &op, double omega, const double *e, const double *uin,
                           const double *f, double *uout, int m, const int *done, hipStream_t s);
// Most partial sums of a launch_rbc_pre on a side-m level.
int rbc_pre_partials(int m);

// ---- LDS-resident tail (rbc_tail.hip): the standard and rotated levels of side 65 and 33
// (or 33 alone) and the 17^2 coarsest level, solved by sine transforms.
struct RbcTailArgs {
  RbcOp op[4];        // side 65 standard and rotated (top 65 only), side 33 standard and rotated
  double om[4];       // omega / c0 of each
  int gamma, nu1, nu2;
  int visits;         // visits of the top level in a row
  int zero;           // 1: the top level's iterate is zero (u is not read)
  const double *f;    // the top level's right-hand side and iterate, side x side
  double *u;
  const double *dst;  // rbc_tail_table, on the device
  const int *done;    // may be null
};
// The sine table (15 x 15) and the 225 per-mode factors of the 17^2 level's operator.
std::vector<double> rbc_tail_table(const RbcOp &op);
size_t rbc_tail_lds(int top);
hipError_t rbc_tail_prepare(int top);
hipError_t launch_rbc_tail(int top, const RbcTailArgs &a, hipStream_t s);

}  // namespace mgk
