// Fock operator y = A_F x (equation Preconditioner, Appendix C working
// equations extended to singles), f_ov-free part, in two launches:
//
//   y_ij^ab = sum_c f_ac x_ij^cb + sum_c x_ij^ac f_cb      (virtual kernel)
//             - sum_k f_ki x_kj^ab - sum_k f_kj x_ik^ab     (occupied kernel)
//   y_i^a   = sum_c f_ac x_i^c - sum_k f_ki x_k^a          (occupied kernel)
//
// f_oo and f_vv are symmetric (any orthogonal gauge). Vectors are packed as
// [x1 (o*v) | x2 (o*o*v*v)], x1[i][a], x2[i][j][a][b].
#pragma once

#include "common.hpp"

namespace pnk {

constexpr int kFockOpMaxOcc = 31;  // the occupied kernel stages o^2 slices in LDS

struct FockOp {
  int o = 0, v = 0;
  const double* f_oo = nullptr;
  const double* f_vv = nullptr;
  // set by fock_op_plan
  int bm = 0, tiles = 0;    // virtual kernel: bm x bm blocks, tiles per pair
  int ch = 0, nchunks = 0;  // occupied kernel: ch (ab) elements per workgroup
  int nsingles = 0;         // ... plus workgroups of 16 singles each
  int64_t nparts() const { return (int64_t)nchunks + nsingles; }
};

// Picks the launch shapes; false when these kernels do not apply (o too
// large) and the caller must use the general path.
bool fock_op_plan(FockOp& op);

// y = A_F x (y must not alias x)
void fock_op_apply(const FockOp& op, const double* x1, const double* x2, double* y1, double* y2, hipStream_t s);

}  // namespace pnk
