// Small CCSD-specific kernels (HBM or launch-latency bound).

#include "cc_kernels.hpp"
#include "tensor_ops.hpp"

namespace pnk {
namespace {

inline int grid_for(int64_t n, int cap = 4096) {
  int64_t g = ceil_div(n, 256);
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

__global__ void assemble_fock_kernel(int o, int v, const double* f_oo, const double* f_ov, const double* f_vv,
                                     double* f) {
  const int n = o + v;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n * n; e += gridDim.x * blockDim.x) {
    const int p = e / n, q = e % n;
    double x;
    if (p < o && q < o) x = f_oo[p * o + q];
    else if (p < o) x = f_ov[p * v + (q - o)];
    else if (q < o) x = f_ov[q * v + (p - o)];
    else x = f_vv[(p - o) * v + (q - o)];
    f[e] = x;
  }
}

__global__ void extract_occ_rows_kernel(int naux, int o, int n, const double* L, double* Lo) {
  const int64_t total = (int64_t)naux * o * n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t P = e / ((int64_t)o * n);
    const int64_t r = e % ((int64_t)o * n);
    Lo[e] = L[P * n * n + r];
  }
}

__global__ void extract_blocks_kernel(int naux, int o, int v, const double* L, const double* h, double* Loo,
                                      double* Lov, double* Lvo, double* Lvv) {
  const int n = o + v;
  const int64_t nn = (int64_t)n * n;
  const int64_t total = (int64_t)(naux + 1) * nn;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t P = e / nn;
    const int r = (int)(e % nn);
    const int p = r / n, q = r % n;
    const double x = (P < naux) ? L[e] : h[r];
    if (p < o && q < o) Loo[(P * o + p) * o + q] = x;
    else if (p < o) Lov[(P * o + p) * v + (q - o)] = x;
    else if (q < o) Lvo[(P * o + q) * v + (p - o)] = x;
    else Lvv[(P * v + (p - o)) * v + (q - o)] = x;
  }
}

__global__ void trace_slices_kernel(int nslices, int o, const double* X, double* D) {
  for (int P = blockIdx.x * blockDim.x + threadIdx.x; P < nslices; P += gridDim.x * blockDim.x) {
    double acc = 0.0;
    const double* x = X + (int64_t)P * o * o;
    for (int k = 0; k < o; ++k) acc += x[k * o + k];
    D[P] = acc;
  }
}

__global__ void trace_occ_kernel(int naux, int o, int n, const double* L, double* d) {
  for (int P = blockIdx.x * blockDim.x + threadIdx.x; P < naux; P += gridDim.x * blockDim.x) {
    double acc = 0.0;
    const double* x = L + (int64_t)P * n * n;
    for (int k = 0; k < o; ++k) acc += x[k * n + k];
    d[P] = acc;
  }
}

__global__ __launch_bounds__(256) void energy_stage1(int o, int v, const double* __restrict__ f_ov,
                                                     const double* __restrict__ Itil, const double* __restrict__ t1,
                                                     const double* __restrict__ t2, double* partials) {
  __shared__ double sm[256];
  const int64_t ov = (int64_t)o * v;
  const int64_t N2 = ov * ov;
  const int64_t vv = (int64_t)v * v;
  double acc = 0.0;
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < N2; e += (int64_t)gridDim.x * 256) {
    const int64_t ij = e / vv;
    const int ab = (int)(e % vv);
    const int i = (int)(ij / o), j = (int)(ij % o);
    const int a = ab / v, b = ab % v;
    acc += Itil[e] * (t2[e] + t1[i * v + a] * t1[j * v + b]);
  }
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < ov; e += (int64_t)gridDim.x * 256)
    acc += 2.0 * f_ov[e] * t1[e];
  sm[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(256) void sum_partials(int nparts, const double* partials, double* out) {
  __shared__ double sm[256];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 256) acc += partials[i];
  sm[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sm[0];
}

__global__ void jacobi_kernel(int o, int v, const double* __restrict__ f_oo, const double* __restrict__ f_vv,
                              double shift, const double* __restrict__ r, double* __restrict__ t,
                              double* __restrict__ step) {
  const int64_t ov = (int64_t)o * v;
  const int64_t N = ov + ov * ov;
  const int64_t vv = (int64_t)v * v;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < N; e += (int64_t)gridDim.x * blockDim.x) {
    double D;
    if (e < ov) {
      const int i = (int)(e / v), a = (int)(e % v);
      D = f_vv[a * v + a] - f_oo[i * o + i];
    } else {
      const int64_t q = e - ov;
      const int64_t ij = q / vv;
      const int ab = (int)(q % vv);
      const int i = (int)(ij / o), j = (int)(ij % o);
      const int a = ab / v, b = ab % v;
      D = f_vv[a * v + a] + f_vv[b * v + b] - f_oo[i * o + i] - f_oo[j * o + j];
    }
    const double st = -r[e] / (D + shift);
    t[e] += st;
    if (step) step[e] = st;
  }
}

__global__ void scale_inv_kernel(int64_t n, const double* __restrict__ x, const double* __restrict__ s,
                                 double* __restrict__ y) {
  const double inv = *s != 0.0 ? 1.0 / *s : 0.0;  // a zero vector stays zero
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = x[i] * inv;
}

__device__ inline int64_t upair(int x, int y, int n) {  // x <= y
  return (int64_t)x * n - (int64_t)x * (x - 1) / 2 + (y - x);
}
__device__ inline int64_t spair(int x, int y, int n) {  // x < y
  return (int64_t)x * (n - 1) - (int64_t)x * (x - 1) / 2 + (y - x - 1);
}
// Occupied pairs of the ladder, i <= j: the n(n-1)/2 pairs i < j first (in
// spair order), then the n diagonal pairs. The antisymmetric ladder
// vanishes on i = j for pair-symmetric t2, so its product runs over the
// first n(n-1)/2 rows only.
__device__ inline int64_t opair(int i, int j, int n) {  // i <= j
  return i < j ? spair(i, j, n) : (int64_t)n * (n - 1) / 2 + i;
}

__global__ void ppl_pack_w_kernel(int v, int a0, int na, const double* __restrict__ Wblk,
                                  const int* __restrict__ pa, const int* __restrict__ pb,
                                  const int* __restrict__ ma, const int* __restrict__ mb, double* __restrict__ S,
                                  int64_t lds, double* __restrict__ A, int64_t lda) {
  const int64_t P2 = (int64_t)v * (v + 1) / 2, P2m = (int64_t)v * (v - 1) / 2;
  const int64_t vv = (int64_t)v * v, v3 = vv * v;
  const int64_t p_lo = upair(a0, a0, v), p_hi = (a0 + na < v) ? upair(a0 + na, a0 + na, v) : P2;
  const int64_t m_lo = (a0 < v - 1) ? spair(a0, a0 + 1, v) : P2m;
  const int64_t m_hi = (a0 + na < v - 1) ? spair(a0 + na, a0 + na + 1, v) : P2m;
  const int64_t ns = (p_hi - p_lo) * P2, nm = (m_hi - m_lo) * P2m;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < ns + nm; e += (int64_t)gridDim.x * blockDim.x) {
    if (e < ns) {
      const int64_t p = p_lo + e / P2, q = e % P2;
      const int a = pa[p], b = pb[p], c = pa[q], d = pb[q];
      const double* w = Wblk + (a - a0) * v3 + (int64_t)b * vv;
      S[p * lds + q] = (a == b ? 0.5 : 1.0) * (w[(int64_t)c * v + d] + w[(int64_t)d * v + c]);
    } else {
      const int64_t f = e - ns;
      const int64_t p = m_lo + f / P2m, q = f % P2m;
      const int a = ma[p], b = mb[p], c = ma[q], d = mb[q];
      const double* w = Wblk + (a - a0) * v3 + (int64_t)b * vv;
      A[p * lda + q] = w[(int64_t)c * v + d] - w[(int64_t)d * v + c];
    }
  }
}

// Pair (x <= y) number k of n, in upair order.
__device__ inline void upair_inverse(int k, int n, int* x, int* y) {
  int r = 0;
  while (k >= n - r) {
    k -= n - r;
    ++r;
  }
  *x = r;
  *y = r + k;
}

// Every layout of the doubles that the contractions read, from one pass over
// t: a workgroup takes the 32 x 32 tiles (A, B) and (B, A), A <= B, of one
// pair (i, j), so each element meets its exchange partner t_ij^ba in LDS and
// all writes run along rows. HBM-bound: at o = 20, v = 180 (104 MB per
// array) 72 us with one read and three written, 200 us with seven, in place of
// a pass per layout and the ladder's packing (ten launches, 0.46 ms).
constexpr int kT = 32;

__global__ __launch_bounds__(256) void amp_layouts_kernel(int o, int v, int tiles, AmpLayouts p) {
  __shared__ double s1[kT][kT + 1], s2[kT][kT + 1];
  int A, B;
  upair_inverse(blockIdx.x, tiles, &A, &B);
  const int ij = blockIdx.y, i = ij / o, j = ij % o;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t vv = (int64_t)v * v;
  const double* __restrict__ t = p.t + ij * vv;
  const bool same = A == B;
#pragma unroll
  for (int r = 0; r < kT; r += 8) {
    const int a = A * kT + ty + r, b = B * kT + tx;
    if (a < v && b < v) s1[ty + r][tx] = t[(int64_t)a * v + b];
    const int c = B * kT + ty + r, d = A * kT + tx;
    if (!same && c < v && d < v) s2[ty + r][tx] = t[(int64_t)c * v + d];
  }
  __syncthreads();
  const double(*sx)[kT + 1] = same ? s1 : s2;
  const int64_t P2 = (int64_t)v * (v + 1) / 2, P2m = (int64_t)v * (v - 1) / 2;
  const int64_t pij = i <= j ? opair(i, j, o) : 0;
  if (blockIdx.x == 0 && i <= j) {  // the rows' padding
    if (P2 + threadIdx.x < p.ldp) p.Tp[pij * p.ldp + P2 + threadIdx.x] = 0.0;
    if (i < j && P2m + threadIdx.x < p.ldm) p.Tm[pij * p.ldm + P2m + threadIdx.x] = 0.0;
  }
  // x = t_ij^ab, y = t_ij^ba
  auto emit = [&](int a, int b, double x, double y) {
    const int64_t m = (((int64_t)i * v + a) * o + j) * v + b;
    const double u = 2.0 * x - y;
    p.Tsia[m] = y;
    p.Uia[m] = u;
    if (p.U) {
      p.Tia[m] = x;
      const int64_t q = ij * vv + (int64_t)a * v + b;
      p.U[q] = u;
      p.Uklca[q] = 2.0 * y - x;
      p.Uail[(((int64_t)a * o + i) * o + j) * v + b] = u;
    }
    if (i <= j && a <= b) {
      p.Tp[pij * p.ldp + upair(a, b, v)] = a == b ? p.diag * x : 0.5 * (x + y);
      if (i < j && a < b) p.Tm[pij * p.ldm + spair(a, b, v)] = 0.5 * (x - y);
    }
  };
#pragma unroll
  for (int r = 0; r < kT; r += 8) {
    const int a = A * kT + ty + r, b = B * kT + tx;
    if (a < v && b < v) emit(a, b, s1[ty + r][tx], sx[tx][ty + r]);
  }
  if (same) return;
#pragma unroll
  for (int r = 0; r < kT; r += 8) {
    const int b = B * kT + ty + r, a = A * kT + tx;
    if (a < v && b < v) emit(b, a, s2[ty + r][tx], s1[tx][ty + r]);
  }
}

// The doubles residual from its parts,
//   R_ij^ab (+)= E[(i,a)][(j,b)] + P_ij^ab V_ij^ab + ladder_ij^ab,
//   V_ij^ab = X[i][j][a][b] + T[(i,a)][(j,b)] + S[(j,a)][(i,b)] + w S[(i,a)][(j,b)],
// the ladder unpacked from its symmetric and antisymmetric combinations (E
// may be null). A workgroup takes the tiles (A, B), (B, A), A <= B, of (i, j)
// and (j, i), i <= j: each part is read once, along rows, transposed
// partners meet in LDS. HBM-bound: at o = 20, v = 180 119 us for four arrays
// of 104 MB read (S from cache where it is read again) and one written, in place
// of two permutations into X, one into R, the unpacking and the pair sum (five
// launches, 0.40 ms).
__global__ __launch_bounds__(256) void doubles_sum_kernel(int o, int v, int tiles, DoublesParts p) {
  __shared__ double st[kT][kT + 1], sx[kT][kT + 1];
  int A, B, i, j;
  upair_inverse(blockIdx.x, tiles, &A, &B);
  upair_inverse(blockIdx.y, o, &i, &j);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t vv = (int64_t)v * v;
  const int64_t pij = opair(i, j, o);
  const bool offd = i < j;  // the antisymmetric part has rows i < j only
  auto ia = [&](int x, int a, int y, int b) { return (((int64_t)x * v + a) * o + y) * v + b; };
  auto ij = [&](int x, int y, int a, int b) { return ((int64_t)x * o + y) * vv + (int64_t)a * v + b; };
  auto V = [&](int x, int y, int a, int b) {
    double s = p.X[ij(x, y, a, b)] + p.T[ia(x, a, y, b)] + p.S[ia(y, a, x, b)];
    if (p.w != 0.0) s += p.w * p.S[ia(x, a, y, b)];
    return s;
  };
  // tiles (P, Q) of (i, j) and (Q, P) of (j, i)
  auto half = [&](int P, int Q, bool first) {
    double d[kT / 8], r1[kT / 8], r2[kT / 8];
#pragma unroll
    for (int q = 0; q < kT / 8; ++q) {
      const int a = P * kT + ty + 8 * q, b = Q * kT + tx;
      d[q] = r1[q] = 0.0;
      if (a < v && b < v) {
        d[q] = V(i, j, a, b);
        if (p.add) r1[q] = p.R[ij(i, j, a, b)];
        if (p.E) r1[q] += p.E[ia(i, a, j, b)];
      }
      const int c = Q * kT + ty + 8 * q, e = P * kT + tx;
      r2[q] = 0.0;
      if (c < v && e < v) {
        st[ty + 8 * q][tx] = V(j, i, c, e);
        if (p.add) r2[q] = p.R[ij(j, i, c, e)];
        if (p.E) r2[q] += p.E[ia(j, c, i, e)];
      }
    }
    double x[kT / 8];  // the ladder
    if (first) {
#pragma unroll
      for (int q = 0; q < kT / 8; ++q) {
        const int a = P * kT + ty + 8 * q, b = Q * kT + tx;
        double xs = 0.0, xa = 0.0;
        if (a < v && b < v) {
          const int lo = min(a, b), hi = max(a, b);
          xs = p.Rp[pij * p.ldp + upair(lo, hi, v)];
          if (offd && a != b) xa = p.Rm[pij * p.ldm + spair(lo, hi, v)];
          if (a > b) xa = -xa;
        }
        x[q] = xs + xa;
        sx[ty + 8 * q][tx] = xs - xa;
      }
    } else {
#pragma unroll
      for (int q = 0; q < kT / 8; ++q) x[q] = sx[tx][ty + 8 * q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kT / 8; ++q) {
      const int a = P * kT + ty + 8 * q, b = Q * kT + tx;
      d[q] += st[tx][ty + 8 * q];
      d[q] += x[q];
      if (a < v && b < v) p.R[ij(i, j, a, b)] = r1[q] + d[q];
    }
    if (i == j && P == Q) return;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kT / 8; ++q) st[ty + 8 * q][tx] = d[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kT / 8; ++q) {
      const int c = Q * kT + ty + 8 * q, e = P * kT + tx;
      if (c < v && e < v) p.R[ij(j, i, c, e)] = r2[q] + st[tx][ty + 8 * q];
    }
  };
  half(A, B, true);
  if (i < j && A < B) {
    __syncthreads();
    half(B, A, false);
  }
}

// The (k,b) and (k,l) columns of the ladder's matrices: 32 rows of W by 32
// pairs (c, d) through LDS, read along d and written along the rows' index.
template <bool ANTI>
__global__ __launch_bounds__(256) void ladder_columns_kernel(int v, int64_t pairs, int cols, int o,
                                                             const double* __restrict__ W, const int* __restrict__ pc,
                                                             const int* __restrict__ pd, double* __restrict__ S,
                                                             int64_t lds) {
  __shared__ double st[kT][kT + 1];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int64_t q0 = (int64_t)blockIdx.x * kT;
  const int r0 = blockIdx.y * kT;
  const int64_t q = q0 + tx, vv = (int64_t)v * v;
  if (q < pairs) {
    const int c = pc[q], d = pd[q];
#pragma unroll
    for (int e = 0; e < kT; e += 8) {
      int r = r0 + ty + e;
      if (r >= cols) break;
      if (o > 0) {
        int x, y;
        if (ANTI) {
          upair_inverse(r, o - 1, &x, &y);
          ++y;
        } else {
          upair_inverse(r, o, &x, &y);
        }
        r = x * o + y;
      }
      const double* w = W + r * vv;
      const double a = w[(int64_t)c * v + d], b = w[(int64_t)d * v + c];
      st[ty + e][tx] = ANTI ? a - b : c == d ? a : a + b;
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kT; e += 8) {
    const int64_t p = q0 + ty + e;
    if (p < pairs && r0 + tx < cols) S[p * lds + r0 + tx] = st[tx][ty + e];
  }
}

__global__ void fill_columns_kernel(int64_t rows, double* x, int64_t ld, int cols) {
  const int64_t n = rows * cols;
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256)
    x[e / cols * ld + e % cols] = 0.0;
}

// One thread per element of Z and of Y (with its W and combinations): a few
// megabytes, launch-bound (in place of a permutation, and of the reductions
// of two products split along their 32400-deep sums at v = 180).
__global__ __launch_bounds__(256) void ladder_unpack_kernel(int o, int v, LadderParts p) {
  const LadderLayout l = p.l;
  const int ov = o * v, oo = o * o;
  const int64_t nz = (int64_t)oo * ov, total = nz + (int64_t)oo * oo;
  auto Y = [&](int k, int m, int i, int j) {
    const int lo = min(i, j), hi = max(i, j), kl = min(k, m), kh = max(k, m);
    double y = p.Rp[opair(lo, hi, o) * l.ldp + l.p2 + ov + upair(kl, kh, o)];
    if (i != j && k != m && l.ldm > 0) {
      const double a = p.Rm[opair(lo, hi, o) * l.ldm + l.p2m + ov + spair(kl, kh, o)];
      y += (i < j) == (k < m) ? a : -a;
    }
    return y;
  };
  auto K = [&](int k, int i, int m, int j) { return p.Kilj[(((int64_t)k * o + i) * o + m) * o + j]; };
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    if (e < nz) {
      const int ij = (int)(e / ov), kb = (int)(e % ov), i = ij / o, j = ij % o;
      const int64_t row = opair(min(i, j), max(i, j), o);
      double z = p.Rp[row * l.ldp + l.p2 + kb];
      if (i != j && l.ldm > 0) {
        const double a = p.Rm[row * l.ldm + l.p2m + kb];
        z += i < j ? a : -a;
      }
      p.Z[e] = z;
    } else {
      const int64_t f = e - nz;
      const int kl = (int)(f / oo), ij = (int)(f % oo);
      const int k = kl / o, m = kl % o, i = ij / o, j = ij % o;
      const double y = Y(k, m, i, j), w = y + K(k, i, m, j);
      p.Y[f] = y;
      if (p.Wkl) p.Wkl[f] = w;
      if (i <= j && k <= m) {
        const double w2 = Y(m, k, i, j) + K(m, i, k, j);
        const int64_t row = opair(i, j, o), c = opair(k, m, o);
        p.Wp[row * l.o2k + c] = k == m ? w : w + w2;
        if (k == 0 && m == 0 && l.o2k > l.o2) p.Wp[row * l.o2k + l.o2] = 0.0;
        if (i < j && k < m) p.Wm[row * l.o2mk + c] = w - w2;
        if (i < j && k == 0 && m == 0 && l.o2mk > l.o2m) p.Wm[row * l.o2mk + l.o2m] = 0.0;
      }
    }
  }
}

// F = L[naux] + 2 sum_P D_P L[P] of the four dressed blocks, D_P = tr Loo[P],
// or the tangent dL[naux] + 2 sum_P (dD_P L[P] + D_P dL[P]). A workgroup
// takes 64 columns of one block, its four waves every fourth slice; the
// traces of 256 slices at a time are formed by each workgroup for itself.
// HBM-bound (one pass over the blocks, 192 MB at o = 20, v = 180, 600 slices:
// 72 us), in place of a trace, four copies and four one-row products with
// their reductions (thirteen launches, which at o = 4, v = 16 cost 60 us).
constexpr int kSlices = 256;

__global__ __launch_bounds__(256) void fock_sum_kernel(int naux, int o, FockSum p) {
  __shared__ double D[kSlices], dD[kSlices], sm[4][64];
  int blk = blockIdx.x, q = 0;
  while (q < 3 && blk >= (p.n[q] + 63) / 64) blk -= (p.n[q++] + 63) / 64;
  const int n = p.n[q], c = blk * 64 + (threadIdx.x & 63), w = threadIdx.x >> 6;
  const int64_t oo = (int64_t)o * o;
  const bool tangent = p.dLoo != nullptr, in = c < n;
  const double* __restrict__ L = p.L[q] + min(c, n - 1);
  const double* __restrict__ dL = p.dL[q] ? p.dL[q] + min(c, n - 1) : nullptr;
  auto trace = [&](const double* x) {
    double t = 0.0;
#pragma unroll 4
    for (int k = 0; k < o; ++k) t += x[(int64_t)k * (o + 1)];
    return t;
  };
  double acc = 0.0;
  for (int P0 = 0; P0 < naux; P0 += kSlices) {
    const int np = min(kSlices, naux - P0), t = threadIdx.x;
    __syncthreads();
    if (t < np) {
      D[t] = trace(p.Loo + (P0 + t) * oo);
      if (tangent) dD[t] = trace(p.dLoo + (P0 + t) * oo);
      if (p.D && blockIdx.x == 0) p.D[P0 + t] = D[t];
    }
    __syncthreads();
    if (tangent) {
#pragma unroll 8
      for (int s = w; s < np; s += 4) acc += dD[s] * L[(int64_t)(P0 + s) * n];
      if (dL) {
#pragma unroll 8
        for (int s = w; s < np; s += 4) acc += D[s] * dL[(int64_t)(P0 + s) * n];
      }
    } else {
#pragma unroll 8
      for (int s = w; s < np; s += 4) acc += D[s] * L[(int64_t)(P0 + s) * n];
    }
  }
  sm[w][threadIdx.x & 63] = acc;
  __syncthreads();
  if (w != 0 || !in) return;
  acc = sm[0][threadIdx.x] + sm[1][threadIdx.x] + sm[2][threadIdx.x] + sm[3][threadIdx.x];
  const double last = !tangent ? L[(int64_t)naux * n] : dL ? dL[(int64_t)naux * n] : 0.0;
  p.F[q][c] = 2.0 * acc + last;
}

}  // namespace

void ppl_pack_w(int v, int a0, int na, const double* Wblk, const int* pair_a, const int* pair_b, const int* mpair_a,
                const int* mpair_b, double* S, int64_t lds, double* A, int64_t lda, hipStream_t s) {
  const int64_t P2 = (int64_t)v * (v + 1) / 2;
  ppl_pack_w_kernel<<<grid_for(na * (int64_t)v * P2, 32768), 256, 0, s>>>(v, a0, na, Wblk, pair_a, pair_b, mpair_a,
                                                                          mpair_b, S, lds, A, lda);
  PNK_CHECK_LAUNCH();
}
void ladder_columns(int v, int64_t rows, int o, const double* W, const int* pair_a, const int* pair_b,
                    const int* mpair_a, const int* mpair_b, double* S, int64_t lds, double* A, int64_t lda,
                    hipStream_t s) {
  const int64_t p2 = (int64_t)v * (v + 1) / 2, p2m = (int64_t)v * (v - 1) / 2;
  const int64_t cs = o > 0 ? (int64_t)o * (o + 1) / 2 : rows, ca = o > 0 ? (int64_t)o * (o - 1) / 2 : rows;
  ladder_columns_kernel<false><<<dim3((unsigned)ceil_div(p2, kT), (unsigned)ceil_div(cs, kT)), 256, 0, s>>>(
      v, p2, (int)cs, o, W, pair_a, pair_b, S, lds);
  PNK_CHECK_LAUNCH();
  if (p2m == 0 || ca == 0) return;
  ladder_columns_kernel<true><<<dim3((unsigned)ceil_div(p2m, kT), (unsigned)ceil_div(ca, kT)), 256, 0, s>>>(
      v, p2m, (int)ca, o, W, mpair_a, mpair_b, A, lda);
  PNK_CHECK_LAUNCH();
}
void fill_columns(int64_t rows, double* x, int64_t ld, int64_t cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return;
  fill_columns_kernel<<<grid_for(rows * cols), 256, 0, s>>>(rows, x, ld, (int)cols);
  PNK_CHECK_LAUNCH();
}
void ladder_unpack(int o, int v, const LadderParts& p, hipStream_t s) {
  const int64_t oo = (int64_t)o * o;
  ladder_unpack_kernel<<<grid_for(oo * o * v + oo * oo, 8192), 256, 0, s>>>(o, v, p);
  PNK_CHECK_LAUNCH();
}
void amp_layouts(int o, int v, const AmpLayouts& p, hipStream_t s) {
  const int64_t tiles = ceil_div(v, kT), g = tiles * (tiles + 1) / 2;
  PNK_REQUIRE((int64_t)o * o <= 65535 && g < (1ll << 31), "amplitude layouts: extents too large");
  amp_layouts_kernel<<<dim3((unsigned)g, (unsigned)(o * o)), 256, 0, s>>>(o, v, (int)tiles, p);
  PNK_CHECK_LAUNCH();
}
void doubles_sum(int o, int v, const DoublesParts& p, hipStream_t s) {
  const int64_t tiles = ceil_div(v, kT), g = tiles * (tiles + 1) / 2;
  doubles_sum_kernel<<<dim3((unsigned)g, (unsigned)(o * (o + 1) / 2)), 256, 0, s>>>(o, v, (int)tiles, p);
  PNK_CHECK_LAUNCH();
}
void fock_sum(int naux, int o, const FockSum& p, hipStream_t s) {
  int64_t g = 0;
  for (int q = 0; q < 4; ++q) g += ceil_div(p.n[q], 64);
  fock_sum_kernel<<<(unsigned)g, 256, 0, s>>>(naux, o, p);
  PNK_CHECK_LAUNCH();
}

void assemble_fock(int o, int v, const double* f_oo, const double* f_ov, const double* f_vv, double* f,
                   hipStream_t s) {
  const int n = o + v;
  assemble_fock_kernel<<<grid_for((int64_t)n * n), 256, 0, s>>>(o, v, f_oo, f_ov, f_vv, f);
  PNK_CHECK_LAUNCH();
}
void extract_occ_rows(int naux, int o, int n, const double* L, double* Lo, hipStream_t s) {
  extract_occ_rows_kernel<<<grid_for((int64_t)naux * o * n, 16384), 256, 0, s>>>(naux, o, n, L, Lo);
  PNK_CHECK_LAUNCH();
}
void extract_blocks(int naux, int o, int v, const double* L, const double* h, double* Loo, double* Lov,
                    double* Lvo, double* Lvv, hipStream_t s) {
  const int64_t n = o + v;
  extract_blocks_kernel<<<grid_for((naux + 1) * n * n, 16384), 256, 0, s>>>(naux, o, v, L, h, Loo, Lov, Lvo, Lvv);
  PNK_CHECK_LAUNCH();
}
void trace_slices(int nslices, int o, const double* X, double* D, hipStream_t s) {
  trace_slices_kernel<<<grid_for(nslices), 256, 0, s>>>(nslices, o, X, D);
  PNK_CHECK_LAUNCH();
}
void trace_occ(int naux, int o, int n, const double* L, double* d, hipStream_t s) {
  trace_occ_kernel<<<grid_for(naux), 256, 0, s>>>(naux, o, n, L, d);
  PNK_CHECK_LAUNCH();
}
void energy(int o, int v, const double* f_ov, const double* Itil, const double* t1, const double* t2, double* out,
            double* partials, hipStream_t s) {
  energy_stage1<<<kReduceBlocks, 256, 0, s>>>(o, v, f_ov, Itil, t1, t2, partials);
  sum_partials<<<1, 256, 0, s>>>(kReduceBlocks, partials, out);
  PNK_CHECK_LAUNCH();
}
void jacobi_update(int o, int v, const double* f_oo, const double* f_vv, double shift, const double* r, double* t,
                   double* step, hipStream_t s) {
  const int64_t ov = (int64_t)o * v;
  jacobi_kernel<<<grid_for(ov + ov * ov), 256, 0, s>>>(o, v, f_oo, f_vv, shift, r, t, step);
  PNK_CHECK_LAUNCH();
}
void scale_by_inverse(int64_t n, const double* x, const double* s_dev, double* y, hipStream_t s) {
  scale_inv_kernel<<<grid_for(n), 256, 0, s>>>(n, x, s_dev, y);
  PNK_CHECK_LAUNCH();
}

}  // namespace pnk
