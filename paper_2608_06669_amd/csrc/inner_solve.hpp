// The inner solve A_F x = b for symmetric A_F (f_ov = 0): the three-term
// Lanczos form of GMRES (MINRES), run in the orbitals in which the Fock
// blocks are diagonal.
//
// GMRES commutes with an orthogonal change of basis: on the rotated
// right-hand side it takes the same steps, with the same coefficients and
// residual norms, as on the given one. In the eigenvectors of f_oo and f_vv
// the operator is a diagonal d (eps_a + eps_b - eps_i - eps_j on the doubles,
// eps_a - eps_i on the singles), so each element of a Lanczos vector follows
// from the same element of the two before it, and the whole recurrence at an
// element from b there and the scalars alone: v_k = b pi_k(d). A step
// therefore reads b once, rebuilds v_k in registers and reduces; no Lanczos
// vector is stored.
#pragma once

#include "common.hpp"

namespace pnk {

// Eigenvalues and eigenvectors of the Fock blocks on the device. ut_o, ut_v:
// eigenvector k as row k (u_o: as column k); null where the block is diagonal
// already.
struct FockEigen {
  int o = 0, v = 0;
  const double *eps_o = nullptr, *eps_v = nullptr, *ut_o = nullptr, *u_o = nullptr, *ut_v = nullptr;
};

// A vector of the full layout: its singles and its doubles (one array, or two
// of a caller's).
struct VecIn {
  const double *x1 = nullptr, *x2 = nullptr;
};
struct VecOut {
  double *x1 = nullptr, *x2 = nullptr;
};

constexpr int kInnerSegment = 64;  // steps before the recurrence is based anew
constexpr int kInnerCoef = 10;     // scalars kept for each step
constexpr int kInnerState = 16;    // doubles per state slot: two slots, then `fin`
constexpr int kInnerMaxParts = 4096;
// what the host reads after a batch of steps
enum { kInnerFinSteps = 0, kInnerFinRes, kInnerFinBeta, kInnerFinBNorm, kInnerFinRead, kInnerFinTol = kInnerFinRead,
       kInnerFinLimit };

struct InnerSolve {
  FockEigen eig;
  bool packed = false;  // pairs i <= j only (blocks i < j count twice in the sums)
  int blocks = 0, segs = 0;
  int64_t n = 0;        // length of a vector
  // n doubles each: the rotated right-hand side, later v_k; v_{k-1}, w_{k-1},
  // w_{k-2} and x once the recurrence has been based anew
  double *v0 = nullptr, *v1 = nullptr, *w1 = nullptr, *w2 = nullptr, *x = nullptr;
  double *parts = nullptr;  // 2 x 3 kInnerMaxParts: a launch reads one half and writes the other
  double *coef = nullptr;   // kInnerSegment x kInnerCoef
  double *state = nullptr;  // 3 x kInnerState
  double *norm_parts = nullptr;  // 2 x 16 kInnerMaxRows
};
constexpr int kInnerMaxRows = 1024;  // workgroup rows of a launch over pairs
constexpr int64_t kInnerPartsElems =
    2 * 3 * (int64_t)kInnerMaxParts + kInnerSegment * kInnerCoef + 2 * 16 * (int64_t)kInnerMaxRows;

// Sets packed, blocks, segs and n from eig.o and eig.v.
void inner_shape(InnerSolve& q, bool packed);

// v0 = D^1/2 b in the packed layout (the pair-symmetric part of b) or the full
// one, the occupied indices rotated into the eigenvectors of f_oo, D =
// singles_scale on the singles and 1 on the doubles, with the sums of squares
// of both; b is in the full layout. tmp1, tmp2: vectors of the full layout.
// Returns the number of shares of the sums.
int inner_load(const InnerSolve& q, VecIn b, double* tmp1, double* tmp2, double singles_scale, hipStream_t s);
// The state before the first step; rtol ||b|| is the absolute tolerance, and
// `limit` the step the recurrence ends at whatever its residual.
void inner_begin(const InnerSolve& q, int nshares, double rtol, int limit, hipStream_t s);
// Launch `parity` (0, 1, 0, ...) of the recurrence: completes the step whose
// sums the launch before it wrote and writes those of the next. The first
// launch has none to complete, so k steps take k + 1 launches. Once a step
// meets the tolerance or the limit, later launches write nothing.
void inner_step(const InnerSolve& q, int parity, double singles_scale, hipStream_t s);
bool inner_is_step_kernel(const void* func);
// Vectors that fit one workgroup: a segment of kInnerSegment steps, or up to the
// one that meets the tolerance or the limit, in one launch that also stands
// for inner_begin (first segment), inner_finish and its rebase.
bool inner_runs_whole(const InnerSolve& q);
void inner_run(const InnerSolve& q, bool first, int nshares, double rtol, int limit, double singles_scale, hipStream_t s);
// x from the first `steps` of the current segment (of step_base + steps in
// all). With `rebase`, v0, v1, w1, w2 and x are left as the state after them,
// for another kInnerSegment steps, and the launch of `parity` comes next.
void inner_finish(const InnerSolve& q, int steps, bool first_segment, bool rebase, int parity, double singles_scale,
                  hipStream_t s);
// out = D^1/2 x in the full layout, the occupied indices rotated back (from a
// packed solve, x_ji = x_ij^T exactly)
void inner_unload(const InnerSolve& q, double* tmp1, double* tmp2, double singles_scale, VecOut out, hipStream_t s);

// Rotates the virtual indices of `rows` v x v blocks and the singles, in place
// through tmp, into (forward) or out of the eigenvectors of f_vv.
void inner_rotate_vir(const FockEigen& e, bool forward, int64_t rows, double* x, double* tmp, hipStream_t s);

// Host copy of the occupied rotation's position sets for v virtuals: for set
// u and lane l, a[64 u + l], b[64 u + l] is the lane's (a, b) (past v: a
// padding lane) and lt[64 u + l] the lane holding (b, a). Returns the set
// count, or -1 when v < 1 or cap (elements per array) is too small.
int inner_set_positions(int v, int* a, int* b, int* lt, int64_t cap);

}  // namespace pnk
