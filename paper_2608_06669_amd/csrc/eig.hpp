// Eigenvalues of a small real upper Hessenberg matrix on the host (the
// Ritz values of an Arnoldi process), and the eigendecomposition of a
// symmetric one (the Fock blocks).
#pragma once

namespace pnk {

// H: m x m, row-major, upper Hessenberg (entries below the subdiagonal are
// ignored). Writes the m eigenvalues to re[], im[] (no particular order).
// Returns false if the iteration did not converge.
bool hessenberg_eigenvalues(const double* H, int m, double* re, double* im);

// F = U diag(eps) U^T for the n x n row-major symmetric F (its symmetric part
// is taken). ut[k n + a] = U[a][k]: eigenvector k as row k. An exactly diagonal
// F gives its diagonal and the identity, *diagonal = true. Returns false for a
// matrix that is not finite or if the iteration did not converge.
bool symmetric_eigen(const double* F, int n, double* eps, double* ut, bool* diagonal);

}  // namespace pnk
