// Small problem-specific kernels of the CCSD path (bandwidth or latency
// bound): integral block extraction, Fock assembly, traces, the energy
// reduction and the Jacobi update.
#pragma once

#include "common.hpp"

namespace pnk {

// f[n][n] from f_oo [o][o], f_ov [o][v], f_vv [v][v] (f_vo = f_ov^T)
void assemble_fock(int o, int v, const double* f_oo, const double* f_ov, const double* f_vv, double* f,
                   hipStream_t s);
// Lo[P][k][q] = L[P][k][q] for k < o (rows of the occupied orbitals)
void extract_occ_rows(int naux, int o, int n, const double* L, double* Lo, hipStream_t s);
// Blocks of the np = naux + 1 slices [L[0..naux-1]; h]: oo [np][o][o],
// ov [np][o][v], vo transposed [np][o][v], vv [np][v][v]
void extract_blocks(int naux, int o, int v, const double* L, const double* h, double* Loo, double* Lov,
                    double* Lvo, double* Lvv, hipStream_t s);
// D[P] = sum_k X[P][k][k] for P < nslices, X of shape [.][o][o]
void trace_slices(int nslices, int o, const double* X, double* D, hipStream_t s);
// d[P] = sum_{k<o} L[P][k][k], L of shape [naux][n][n]
void trace_occ(int naux, int o, int n, const double* L, double* d, hipStream_t s);
// E = 2 sum f_ov t1 + sum_ijab Itil (t2 + t1_ia t1_jb) -> out (device), deterministic
void energy(int o, int v, const double* f_ov, const double* Itil, const double* t1, const double* t2, double* out,
            double* partials, hipStream_t s);
// t <- t - r / (D + shift) with Jacobi denominators from diag(f_oo), diag(f_vv);
// e = -r / (D + shift) is written to `step` when it is not null
void jacobi_update(int o, int v, const double* f_oo, const double* f_vv, double shift, const double* r, double* t,
                   double* step, hipStream_t s);
// Symmetry-adapted particle-particle ladder. Pairs a <= b are numbered
// row-major over the upper triangle (p), pairs a < b likewise (p'), and
// occupied pairs i <= j likewise; pair_a/pair_b map a packed index back.
// S[p][q] = W_ab,cd + W_ab,dc (halved for a = b) and A[p'][q'] = W_ab,cd -
// W_ab,dc (row lengths lds, lda) for the rows whose a lies in [a0, a0 + na);
// Wblk[a - a0][b][c][d] = (ac|bd).
void ppl_pack_w(int v, int a0, int na, const double* Wblk, const int* pair_a, const int* pair_b,
                const int* mpair_a, const int* mpair_b, double* S, int64_t lds, double* A, int64_t lda, hipStream_t s);
// S[q][r] = W_r,cd + W_r,dc (half of it for c = d), A[q'][r] = W_r,cd - W_r,dc
// from W[r][c][d], r < rows. With o > 0 the rows of W are pairs (k, l) of o
// and the columns run over k <= l (S, row-major) and k < l (A).
void ladder_columns(int v, int64_t rows, int o, const double* W, const int* pair_a, const int* pair_b,
                    const int* mpair_a, const int* mpair_b, double* S, int64_t lds, double* A, int64_t lda,
                    hipStream_t s);
// x[r][c] = 0, r < rows, c < cols, row length ld
void fill_columns(int64_t rows, double* x, int64_t ld, int64_t cols, hipStream_t s);

// Lengths of the packed ladder: pairs of virtuals c <= d (p2) and c < d (p2m),
// of occupied i <= j (o2) and i < j (o2m). T+ and T- have rows of p2k and p2mk
// and o2k, o2mk of them (zero past the pairs); S, R+ (ldp) and A, R- (ldm) have
// columns for the pairs, for (k,b) and for k <= l (k < l), then padding.
struct LadderLayout {
  int64_t p2, p2m, o2, o2m, p2k, p2mk, ldp, ldm, o2k, o2mk;
};
// From the (k,b) and (k,l) columns of R+, R-: Z[(i,j)][(k,b)] = sum_cd (kc|bd)
// t_ij^cd, Y[(k,l)][(i,j)] = sum_cd (kc|ld) t_ij^cd, W_klij = Kilj[(k,i)][(l,j)] +
// Y and its combinations Wp[ij][kl] = W_klij + W_lkij (W_kkij once), rows i <= j
// and o2k columns, Wm = W_klij - W_lkij, i < j, k < l. Wkl (all W) may be null.
struct LadderParts {
  LadderLayout l;
  const double *Rp, *Rm, *Kilj;
  double *Z, *Y, *Wp, *Wm, *Wkl;
};
void ladder_unpack(int o, int v, const LadderParts& p, hipStream_t s);

// Layouts of doubles t[i][j][a][b] (u = 2 t_ij^ab - t_ij^ba):
struct AmpLayouts {
  const double* t;
  double *Tsia, *Uia;  // [(i,a)][(j,b)]: t_ij^ba, u_ij^ab
  // Tp[ij][q] = (t_ij^cd + t_ij^dc)/2 (c < d) or diag t_ij^cc (c = d), i <= j;
  // Tm[ij][q'] = (t_ij^cd - t_ij^dc)/2, i < j; rows zero past the pairs
  double *Tp, *Tm;
  int64_t ldp, ldm;
  double diag;
  // (all null: not wanted) [(i,a)][(j,b)]: t_ij^ab; [i][j][a][b]: u_ij^ab, u_ij^ba; [a][i][j][b]: u_ij^ab
  double *Tia, *U, *Uklca, *Uail;
};
void amp_layouts(int o, int v, const AmpLayouts& p, hipStream_t s);

// R[i][j][a][b] (+)= E[(i,a)][(j,b)] + V_ij^ab + V_ji^ba + sum_cd (ac|bd) t_ij^cd,
// V_ij^ab = X[i][j][a][b] + T[(i,a)][(j,b)] + S[(j,a)][(i,b)] + w S[(i,a)][(j,b)],
// the ladder rebuilt from Rp = Tp S, Rm = Tm A; E may be null.
struct DoublesParts {
  const double *X, *T, *S, *Rp, *Rm, *E;
  int64_t ldp, ldm;  // row lengths of Rp, Rm
  double w;
  bool add;  // to what R holds (else R is written)
  double* R;
};
void doubles_sum(int o, int v, const DoublesParts& p, hipStream_t s);

// F[q][c] = L[q][naux][c] + 2 sum_P D_P L[q][P][c], c < n[q], P < naux, D_P = tr
// Loo[P] (also written to D unless null). With dLoo, the tangent instead,
// dL[q][naux][c] + 2 sum_P (dD_P L[q][P][c] + D_P dL[q][P][c]); null dL[q]: zero.
struct FockSum {
  const double *Loo, *dLoo;
  int n[4];
  const double *L[4], *dL[4];
  double* F[4];
  double* D;
};
void fock_sum(int naux, int o, const FockSum& p, hipStream_t s);

// y = x / *s_dev (the divisor stays on the device; y = 0 when it is 0)
void scale_by_inverse(int64_t n, const double* x, const double* s_dev, double* y, hipStream_t s);

}  // namespace pnk
