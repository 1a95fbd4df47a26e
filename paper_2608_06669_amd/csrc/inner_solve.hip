// Lanczos form of GMRES in the eigenvectors of the Fock blocks (see
// inner_solve.hpp).

#include "inner_solve.hpp"

#include <algorithm>
#include <cmath>

#include "block_sum.hpp"
#include "gemm.hpp"

namespace pnk {
namespace {

// state slot: beta_k, the two last Givens rotations, phibar, the flags, and
// how many steps of the segment are complete
enum { kSBeta = 0, kSC2, kSS2, kSC1, kSS1, kSPhiBar, kSDone, kSPending, kSCount, kSScale, kSBased, kSTotal, kSSk, kSSp };
// a step's scalars: v_{j+1} = (d ib + c1) v_j + c2 v_{j-1}; w_j = (v_j - delta
// w_{j-1} - eps w_{j-2}) ir; x += phi w_j. With v_j = s_j z_j and s_{j+1} = -c2
// s_{j-1} (s_0 = s_{-1} = 1) the recurrence is z_{j+1} = (d A + B) z_j -
// z_{j-1}, two operations for each element and step in place of three.
enum { kCA = 0, kCB, kCS, kCIb, kCC1, kCC2, kCDelta, kCEps, kCIr, kCPhi };

struct Args {
  int o, v, blocks, npair, segs;  // blocks: workgroup rows; npair: v x v blocks of a vector
  int parity;
  const double *eps_o, *eps_v;
  const double* v0;
  const double* v1;
  const double* part_in;
  double* part_out;
  double* coef;
  double* state;
  double sscale;
};

__device__ inline void decode_pair(int pr, int o, bool packed, int& i, int& j) {
  if (!packed) {
    i = pr / o;
    j = pr - i * o;
    return;
  }
  i = 0;
  while (pr >= o - i) {
    pr -= o - i;
    ++i;
  }
  j = i + pr;
}

// Block y of a vector: v x v elements of pair y, or the singles (y = npair).
struct Block {
  bool singles;
  int len;
  int64_t base;
  double e0, w;  // e_i + e_j (doubles); weight in the sums
};
__device__ inline Block block_of(const Args& p, int y, bool packed) {
  Block b;
  const int64_t vv = (int64_t)p.v * p.v, ov = (int64_t)p.o * p.v;
  b.singles = y == p.npair;
  if (b.singles) {
    b.len = (int)ov;
    b.base = 0;
    b.e0 = 0.0;
    b.w = 1.0;
  } else {
    int i, j;
    decode_pair(y, p.o, packed, i, j);
    b.len = (int)vv;
    b.base = ov + y * vv;
    b.e0 = p.eps_o[i] + p.eps_o[j];
    b.w = packed && i != j ? 2.0 : 1.0;
  }
  return b;
}

// E elements q, q + 256, ... of block b: row r[e] = q / v, column c[e] (past the
// block: its last element)
template <int E>
struct Places {
  int q[E], r[E], c[E];
  __device__ inline Places(const Args& p, const Block& b, int q0) {
    const int dr = 256 / p.v, dc = 256 - dr * p.v;
    int rr = q0 / p.v, cc = q0 - rr * p.v;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      q[e] = min(q0 + 256 * e, b.len - 1);
      const bool in = q0 + 256 * e < b.len;
      r[e] = in ? rr : b.len / p.v - 1;
      c[e] = in ? cc : p.v - 1;
      rr += dr;
      cc += dc;
      if (cc >= p.v) {
        cc -= p.v;
        ++rr;
      }
    }
  }
};
// the operator's diagonal there; ev: eps_v in LDS
__device__ inline double diagonal(const Args& p, const Block& b, const double* ev, int r, int c) {
  return b.singles ? p.sscale * (ev[c] - p.eps_o[r]) : ev[r] + ev[c] - b.e0;
}

// One step (see inner_step). Bound: at o = 20, v = 180 (7.0 M elements) the
// read of b, 56 MB, and 2 FP64 operations per element for every step behind
// it; E elements per thread run side by side, since each one's recurrence is a
// dependent chain. The scalars of the steps behind and eps_v come from LDS
// (read from memory inside the chain, a step took 27 us plus 2 us for each
// step behind; now 15 us plus 0.65). Each workgroup adds the partial sums of the launch
// before in the same fixed order, so all take the same scalars and no
// reduction needs a launch of its own.
template <bool PACKED, int E>
__global__ __launch_bounds__(256) void inner_step_kernel(Args p) {
  const double* __restrict__ st = p.state + p.parity * kInnerState;
  double* __restrict__ stn = p.state + (1 - p.parity) * kInnerState;
  double* __restrict__ fin = p.state + 2 * kInnerState;
  const bool lead = blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0;
  extern __shared__ __attribute__((aligned(16))) double ev[];  // eps_v
  __shared__ __attribute__((aligned(16))) double cf[kInnerSegment + 1][2];  // A, B of the steps behind
  __shared__ double sm[3][4];
  const int tid = threadIdx.x;
  const int nparts = p.blocks * p.segs;
  // the first batch's elements and the shares of the launch before are on
  // their way while the state is read
  int y = blockIdx.y;
  Block b = block_of(p, y, PACKED);
  auto span = [&](int* q0, int* q1) {  // this workgroup's part of block b
    const int per = (b.len + p.segs - 1) / p.segs;
    *q0 = blockIdx.x * per;
    *q1 = min(b.len, *q0 + per);
  };
  int qb, q1;
  span(&qb, &q1);
  double raw[E];
  auto fetch = [&]() {
#pragma unroll
    for (int e = 0; e < E; ++e) raw[e] = p.v0[b.base + min(qb + tid + 256 * e, b.len - 1)];
  };
  fetch();
  double r[3] = {0.0, 0.0, 0.0};
  for (int q = tid; q < nparts; q += 256) {
    r[0] += p.part_in[q];
    r[1] += p.part_in[nparts + q];
    r[2] += p.part_in[2 * nparts + q];
  }
  if (st[kSDone] != 0.0) {
    if (lead) stn[kSDone] = 1.0;
    return;
  }
  int k = (int)st[kSCount];
  const double scale = st[kSScale];
  const bool based = st[kSBased] != 0.0;
  double beta = st[kSBeta];
  const bool pending = st[kSPending] != 0.0;
  for (int q = tid; q < p.v; q += 256) ev[q] = p.eps_v[q];
  for (int q = tid; q < 2 * k; q += 256) cf[q >> 1][q & 1] = p.coef[(q >> 1) * kInnerCoef + (q & 1)];
  double sk = st[kSSk], sp = st[kSSp];  // s_k, s_{k-1}
  if (pending) {
    block_sum256<3>(r, sm);
    // alpha_k = <v_k, p> / <v_k, v_k>, beta_{k+1}^2 = ||p||^2 - alpha <v_k, p>.
    // (Measuring <v_k, v_k> rather than taking it as 1 keeps a rounding error
    // in the norm of v_k from growing from step to step.)
    const double vp = r[0], pp = r[1], vv = r[2];
    const double alpha = vv > 0.0 ? vp / vv : 0.0;
    const double betan = sqrt(fmax(pp - alpha * vp, 0.0));
    const double gc2 = st[kSC2], gs2 = st[kSS2], gc1 = st[kSC1], gs1 = st[kSS1];
    const double eps = gs2 * beta, dbar = gc2 * beta;
    const double delta = gc1 * dbar + gs1 * alpha, gbar = -gs1 * dbar + gc1 * alpha;
    const double rho = hypot(gbar, betan);
    const double c = rho != 0.0 ? gbar / rho : 1.0, sn = rho != 0.0 ? betan / rho : 0.0;
    const double phibar = st[kSPhiBar];
    const double res = fabs(sn * phibar);
    const double ib = betan != 0.0 ? 1.0 / betan : 0.0;
    const double total = st[kSTotal] + 1.0;
    const bool done = res <= fin[kInnerFinTol] || betan == 0.0 || total >= fin[kInnerFinLimit];
    // (beta_k = 0 only before the first step, where z_{-1} = 0)
    const double sn1 = beta * ib != 0.0 ? beta * ib * sp : sk;
    const double ca = ib * (sk / sn1), cb = -alpha * ca;
    if (tid == 0) {
      cf[k][0] = ca;
      cf[k][1] = cb;
    }
    if (lead) {
      double* g = p.coef + k * kInnerCoef;
      g[kCA] = ca;
      g[kCB] = cb;
      g[kCS] = sk;
      stn[kSSk] = sn1;
      stn[kSSp] = sk;
      g[kCIb] = ib;
      g[kCC1] = -alpha * ib;
      g[kCC2] = -beta * ib;
      g[kCDelta] = delta;
      g[kCEps] = eps;
      g[kCIr] = rho != 0.0 ? 1.0 / rho : 0.0;
      g[kCPhi] = c * phibar;
      stn[kSBeta] = betan;
      stn[kSC2] = gc1;
      stn[kSS2] = gs1;
      stn[kSC1] = c;
      stn[kSS1] = sn;
      stn[kSPhiBar] = -sn * phibar;
      stn[kSDone] = done ? 1.0 : 0.0;
      stn[kSPending] = 1.0;
      stn[kSCount] = (double)(k + 1);
      stn[kSScale] = scale;
      stn[kSBased] = st[kSBased];
      stn[kSTotal] = total;
      fin[kInnerFinSteps] = total;
      fin[kInnerFinRes] = res;
      fin[kInnerFinBeta] = betan;
    }
    if (done) return;
    ++k;
    beta = betan;
    sp = sk;
    sk = sn1;
  } else if (lead) {
    for (int q = 0; q < kInnerState; ++q) stn[q] = st[q];
    stn[kSPending] = 1.0;
  }
  __syncthreads();
  double dot = 0.0, nrm = 0.0, vv2 = 0.0;
  while (true) {
    double v[E], u[E], d[E];
    const Places<E> at(p, b, qb + tid);
    const double w = b.w;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const bool in = qb + tid + 256 * e < q1;
      v[e] = in ? scale * raw[e] : 0.0;
      u[e] = in && based ? p.v1[b.base + at.q[e]] : 0.0;
      d[e] = diagonal(p, b, ev, at.r[e], at.c[e]);
    }
    // the next batch of this block, or of the next one this workgroup has
    qb += 256 * E;
    bool more = true;
    while (more && qb >= q1) {
      y += p.blocks;
      more = y <= p.npair;
      if (more) {
        b = block_of(p, y, PACKED);
        span(&qb, &q1);
      }
    }
    if (more) fetch();
#pragma unroll 2
    for (int j = 0; j < k; ++j) {
      const double a = cf[j][0], c = cf[j][1];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double t = (d[e] * a + c) * v[e] - u[e];
        u[e] = v[e];
        v[e] = t;
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const double vk = sk * v[e], x = d[e] * vk - beta * (sp * u[e]);
      dot += w * vk * x;
      nrm += w * x * x;
      vv2 += w * vk * vk;
    }
    if (!more) break;
  }
  r[0] = dot;
  r[1] = nrm;
  r[2] = vv2;
  block_sum256<3>(r, sm);
  if (tid == 0) {
    const int g = blockIdx.y * p.segs + blockIdx.x;
    for (int c = 0; c < 3; ++c) p.part_out[c * nparts + g] = r[c];
  }
}

// x after `steps` steps of the segment. The w recurrence W R = V, x = x_base +
// W phi (R: ir, delta and eps of the steps) is x = x_base + V y + g1 w1 + g2 w2
// with R y = phi, so the recurrence runs once more from its base with one
// multiplication more in each step, and one read and one write of memory.
template <bool PACKED>
__global__ __launch_bounds__(256) void inner_finish_kernel(Args p, int steps, const double* w1, const double* w2,
                                                           double* xo, int first) {
  constexpr int E = 4;
  extern __shared__ __attribute__((aligned(16))) double ev[];
  __shared__ __attribute__((aligned(16))) double cf[kInnerSegment][4];  // A, B, s y
  __shared__ double g[2];
  const int tid = threadIdx.x;
  for (int q = tid; q < p.v; q += 256) ev[q] = p.eps_v[q];
  for (int q = tid; q < 2 * steps; q += 256) cf[q >> 1][q & 1] = p.coef[(q >> 1) * kInnerCoef + (q & 1)];
  if (tid == 0) {
    double y1 = 0.0, y2 = 0.0, d1 = 0.0, e1 = 0.0, e2 = 0.0;  // y, delta, eps of the one and two steps after j
    for (int j = steps - 1; j >= 0; --j) {
      const double* c = p.coef + j * kInnerCoef;
      const double y = (c[kCPhi] - d1 * y1 - e2 * y2) * c[kCIr];
      cf[j][2] = c[kCS] * y;
      y2 = y1;
      y1 = y;
      e2 = e1;
      e1 = c[kCEps];
      d1 = c[kCDelta];
    }
    // (y1 = y_0, y2 = y_1, e2 = eps_1)
    g[0] = -d1 * y1 - e2 * y2;
    g[1] = -e1 * y1;
  }
  __syncthreads();
  const double scale = first ? p.state[p.parity * kInnerState + kSScale] : 1.0;
  for (int y = blockIdx.y; y <= p.npair; y += gridDim.y) {
    const Block b = block_of(p, y, PACKED);
    for (int q = blockIdx.x * 256 * E + tid; q < b.len; q += gridDim.x * 256 * E) {
      const Places<E> at(p, b, q);
      double v[E], u[E], d[E], x[E];
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = scale * p.v0[b.base + at.q[e]];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int64_t z = b.base + at.q[e];
        u[e] = first ? 0.0 : p.v1[z];
        x[e] = first ? 0.0 : xo[z] + g[0] * w1[z] + g[1] * w2[z];
        d[e] = diagonal(p, b, ev, at.r[e], at.c[e]);
      }
#pragma unroll 2
      for (int j = 0; j < steps; ++j) {
        const double a = cf[j][0], c = cf[j][1], yj = cf[j][2];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          x[e] += yj * v[e];
          const double t = (d[e] * a + c) * v[e] - u[e];
          u[e] = v[e];
          v[e] = t;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (q + 256 * e < b.len) xo[b.base + q + 256 * e] = x[e];
    }
  }
}

// The state after a whole segment, as the base of the next: v_k, v_{k-1},
// w_{k-1}, w_{k-2} and x.
template <bool PACKED>
__global__ __launch_bounds__(256) void inner_rebase_kernel(Args p, int steps, double* v0, double* v1, double* w1o,
                                                           double* w2o, double* xo, int first) {
  extern __shared__ __attribute__((aligned(16))) double ev[];
  for (int q = threadIdx.x; q < p.v; q += 256) ev[q] = p.eps_v[q];
  __syncthreads();
  const double scale = first ? p.state[p.parity * kInnerState + kSScale] : 1.0;
  for (int y = blockIdx.y; y <= p.npair; y += gridDim.y) {
    const Block b = block_of(p, y, PACKED);
    for (int q = blockIdx.x * 256 + threadIdx.x; q < b.len; q += gridDim.x * 256) {
      const Places<1> pl(p, b, q);
      const double d = diagonal(p, b, ev, pl.r[0], pl.c[0]);
      const int64_t at = b.base + q;
      double v = scale * v0[at], u = first ? 0.0 : v1[at];
      double w1 = first ? 0.0 : w1o[at], w2 = first ? 0.0 : w2o[at], x = first ? 0.0 : xo[at];
      for (int j = 0; j < steps; ++j) {
        const double* c = p.coef + j * kInnerCoef;
        const double w = (v - c[kCDelta] * w1 - c[kCEps] * w2) * c[kCIr];
        w2 = w1;
        w1 = w;
        x += c[kCPhi] * w;
        const double t = (d * c[kCIb] + c[kCC1]) * v + c[kCC2] * u;
        u = v;
        v = t;
      }
      v0[at] = v;
      v1[at] = u;
      w1o[at] = w1;
      w2o[at] = w2;
      xo[at] = x;
    }
  }
}

// After inner_rebase_kernel: the next launch starts a segment.
__global__ void inner_rebase_state(double* st) {
  if (threadIdx.x) return;
  st[kSCount] = 0.0;
  st[kSScale] = 1.0;
  st[kSBased] = 1.0;
  st[kSSk] = st[kSSp] = 1.0;
}

// v0 = packed D^1/2 sym(b): singles times rs; for i <= j the block (b_ij +
// b_ji^T) / 2 (the pair-symmetric part; b_ji^T staged through LDS). Each
// workgroup writes its shares of ||sym(b)||^2 and ||v0||^2 (blocks of pairs i
// < j counted twice) to parts[g], parts[G + g].
constexpr int kPackTile = 32;
constexpr int kPackBlocksX = 16;  // workgroups per pair block (grid-stride over its tiles)

__global__ __launch_bounds__(256) void inner_pack(int o, int v, VecIn b, double rs, double* __restrict__ xp,
                                                  double* __restrict__ parts) {
  __shared__ double tile[kPackTile][kPackTile + 1];
  __shared__ double sm[2][4];
  const int npair = o * (o + 1) / 2;
  const int64_t vv = (int64_t)v * v, ov = (int64_t)o * v;
  const int tid = threadIdx.x;
  double s_plain = 0.0, s_scaled = 0.0;
  for (int y = blockIdx.y; y <= npair; y += gridDim.y) {
    if (y == npair) {
      for (int64_t e = blockIdx.x * (int64_t)256 + tid; e < ov; e += (int64_t)gridDim.x * 256) {
        const double x = b.x1[e];
        xp[e] = rs * x;
        s_plain += x * x;
        s_scaled += (rs * x) * (rs * x);
      }
      continue;
    }
    int i, j;
    decode_pair(y, o, true, i, j);
    const double w = i == j ? 1.0 : 2.0;
    const double* __restrict__ bij = b.x2 + (int64_t)(i * o + j) * vv;
    const double* __restrict__ bji = b.x2 + (int64_t)(j * o + i) * vv;
    double* __restrict__ out = xp + ov + (int64_t)y * vv;
    const int nt = (v + kPackTile - 1) / kPackTile;
    const int tx = tid % kPackTile, ty = tid / kPackTile;
    for (int tl = blockIdx.x; tl < nt * nt; tl += gridDim.x) {
      const int a0 = (tl / nt) * kPackTile, b0 = (tl % nt) * kPackTile;
      __syncthreads();
      for (int r = ty; r < kPackTile; r += 256 / kPackTile) {  // tile[r][c] = b_ji[b0 + r][a0 + c]
        const int rr = b0 + r, cc = a0 + tx;
        tile[r][tx] = (rr < v && cc < v) ? bji[(int64_t)rr * v + cc] : 0.0;
      }
      __syncthreads();
      for (int r = ty; r < kPackTile; r += 256 / kPackTile) {
        const int a = a0 + r, bb = b0 + tx;
        if (a < v && bb < v) {
          const double x = 0.5 * (bij[(int64_t)a * v + bb] + tile[tx][r]);
          out[(int64_t)a * v + bb] = x;
          s_plain += w * x * x;
          s_scaled += w * x * x;
        }
      }
    }
  }
  double r2[2] = {s_plain, s_scaled};
  block_sum256<2>(r2, sm);
  const int g = blockIdx.y * gridDim.x + blockIdx.x, G = gridDim.x * gridDim.y;
  if (tid == 0) {
    parts[g] = r2[0];
    parts[G + g] = r2[1];
  }
}

// The full layout: v0 = D^1/2 b, with the same shares.
__global__ __launch_bounds__(256) void inner_copy_in(int64_t n, int64_t ov, VecIn b, double rs, double* __restrict__ x,
                                                     double* __restrict__ parts) {
  __shared__ double sm[2][4];
  double r2[2] = {0.0, 0.0};
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
    const double y = e < ov ? b.x1[e] : b.x2[e - ov], z = e < ov ? rs * y : y;
    x[e] = z;
    r2[0] += y * y;
    r2[1] += z * z;
  }
  block_sum256<2>(r2, sm);
  if (threadIdx.x == 0) {
    parts[blockIdx.x] = r2[0];
    parts[gridDim.x + blockIdx.x] = r2[1];
  }
}
__global__ __launch_bounds__(256) void inner_copy_out(int64_t n, int64_t ov, const double* __restrict__ x, double rs,
                                                      VecOut y) {
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256)
    if (e < ov) y.x1[e] = rs * x[e];
    else y.x2[e - ov] = x[e];
}

// x (full layout) = D^1/2 unpack(xp): x_ij = xp_P(i,j) for i <= j, and
// xp_P(j,i)^T (through LDS) for i > j; singles times rs.
__global__ __launch_bounds__(256) void inner_unpack(int o, int v, const double* __restrict__ xp, double rs, VecOut x) {
  __shared__ double tile[kPackTile][kPackTile + 1];
  const int64_t vv = (int64_t)v * v, ov = (int64_t)o * v;
  const int tid = threadIdx.x;
  if ((int)blockIdx.y == o * o) {
    for (int64_t e = blockIdx.x * (int64_t)256 + tid; e < ov; e += (int64_t)gridDim.x * 256) x.x1[e] = rs * xp[e];
    return;
  }
  const int i = blockIdx.y / o, j = blockIdx.y % o;
  auto pair = [&](int a, int b) { return a * o - a * (a - 1) / 2 + (b - a); };  // a <= b
  double* __restrict__ out = x.x2 + (int64_t)blockIdx.y * vv;
  if (i <= j) {
    const double* __restrict__ src = xp + ov + (int64_t)pair(i, j) * vv;
    for (int64_t e = blockIdx.x * (int64_t)256 + tid; e < vv; e += (int64_t)gridDim.x * 256) out[e] = src[e];
    return;
  }
  const double* __restrict__ src = xp + ov + (int64_t)pair(j, i) * vv;  // x_ij = x_ji^T
  const int nt = (v + kPackTile - 1) / kPackTile;
  const int tx = tid % kPackTile, ty = tid / kPackTile;
  for (int tl = blockIdx.x; tl < nt * nt; tl += gridDim.x) {
    const int a0 = (tl / nt) * kPackTile, b0 = (tl % nt) * kPackTile;
    __syncthreads();
    for (int r = ty; r < kPackTile; r += 256 / kPackTile) {  // tile[r][c] = x_ji[b0 + r][a0 + c]
      const int rr = b0 + r, cc = a0 + tx;
      tile[r][tx] = (rr < v && cc < v) ? src[(int64_t)rr * v + cc] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < kPackTile; r += 256 / kPackTile) {
      const int a = a0 + r, bb = b0 + tx;
      if (a < v && bb < v) out[(int64_t)a * v + bb] = tile[tx][r];
    }
  }
}

// ||b|| and ||v0|| from the shares (summed in a fixed order by one
// workgroup), and the state before the first step: v_1 = v0 / ||v0||, no sums
// pending.
__global__ __launch_bounds__(256) void inner_begin_kernel(const double* __restrict__ parts, int nparts, double* state,
                                                          double rtol, double limit) {
  __shared__ double sm[2][4];
  double r[2] = {0.0, 0.0};
  for (int k = threadIdx.x; k < nparts; k += 256) {
    r[0] += parts[k];
    r[1] += parts[nparts + k];
  }
  block_sum256<2>(r, sm);
  if (threadIdx.x != 0) return;
  const double bn = sqrt(r[0]), bhat = sqrt(r[1]);
  for (int k = 0; k < 3 * kInnerState; ++k) state[k] = 0.0;
  state[kSC2] = 1.0;
  state[kSC1] = 1.0;
  state[kSPhiBar] = bhat;
  state[kSScale] = bhat != 0.0 ? 1.0 / bhat : 0.0;
  state[kSSk] = state[kSSp] = 1.0;
  double* fin = state + 2 * kInnerState;
  fin[kInnerFinRes] = bhat;
  fin[kInnerFinBeta] = 1.0;
  fin[kInnerFinBNorm] = bn;
  fin[kInnerFinTol] = rtol * bn;
  fin[kInnerFinLimit] = limit;
}

// A whole segment of the solve in one workgroup, for vectors of at most
// kRunThreads E elements: the recurrence stays in registers (E elements per
// thread), the three sums of a step go through one barrier and every thread
// forms the scalars for itself; x follows from one more run over them, as in
// inner_finish_kernel. FIRST: b's shares give the norms (as
// inner_begin_kernel); else the state after the segment before it is in
// memory. Bound by the chain of sums and scalars: 1.9 us a step at 2624 elements
// (o = 4, v = 16), 2.6 at 7952 (o = 4, v = 28), where a launch for each step took
// 6.1; 22 steps with the start and x 43 us in place of 157.
constexpr int kRunThreads = 512;

template <bool PACKED, int E>
__global__ __launch_bounds__(kRunThreads) void inner_run_kernel(Args p, int n, bool first, const double* __restrict__ shares,
                                                                int nshares, double rtol, double limit, double* v0,
                                                                double* v1, double* w1o, double* w2o, double* xo) {
  constexpr int NW = kRunThreads / 64;
  __shared__ double sm[2][3][NW];
  __shared__ double cf[kInnerSegment][8];  // A, B, s, delta, eps, 1 / rho, phi; s y
  __shared__ double g[2];
  enum { A = 0, B, S, DELTA, EPS, IR, PHI, Y };
  const int tid = threadIdx.x;
  double* st = p.state;
  double* fin = p.state + 2 * kInnerState;
  int par = 0;
  auto sums = [&](double (&r)[3]) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
      for (int c = 0; c < 3; ++c) r[c] += __shfl_xor(r[c], m, 64);
    if ((tid & 63) == 0)
#pragma unroll
      for (int c = 0; c < 3; ++c) sm[par][c][tid >> 6] = r[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) t += sm[par][c][w];
      r[c] = t;
    }
    par ^= 1;  // (the other half until every thread is past the next barrier)
  };
  // element tid + 512 e: its diagonal, and whether its block counts twice
  double v[E], u[E], d[E];
  uint32_t twice = 0;
  const int ov = p.o * p.v, vv = p.v * p.v;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int q = tid + kRunThreads * e;
    v[e] = u[e] = d[e] = 0.0;
    if (q >= n) continue;
    v[e] = v0[q];
    if (!first) u[e] = v1[q];
    if (q < ov) {
      d[e] = p.sscale * (p.eps_v[q % p.v] - p.eps_o[q / p.v]);
    } else {
      const int f = q - ov, a = f % vv;
      int i, j;
      decode_pair(f / vv, p.o, PACKED, i, j);
      d[e] = p.eps_v[a / p.v] + p.eps_v[a % p.v] - (p.eps_o[i] + p.eps_o[j]);
      if (PACKED && i != j) twice |= 1u << e;
    }
  }
  double beta = 0.0, gc2 = 1.0, gs2 = 0.0, gc1 = 1.0, gs1 = 0.0, phibar, total = 0.0, scale = 1.0, tol;
  if (first) {
    double r[3] = {0.0, 0.0, 0.0};
    for (int k = tid; k < nshares; k += kRunThreads) {
      r[0] += shares[k];
      r[1] += shares[nshares + k];
    }
    sums(r);
    const double bn = sqrt(r[0]), bhat = sqrt(r[1]);
    phibar = bhat;
    scale = bhat != 0.0 ? 1.0 / bhat : 0.0;
    tol = rtol * bn;
    if (tid == 0) fin[kInnerFinBNorm] = bn;
  } else {
    beta = st[kSBeta];
    gc2 = st[kSC2];
    gs2 = st[kSS2];
    gc1 = st[kSC1];
    gs1 = st[kSS1];
    phibar = st[kSPhiBar];
    total = st[kSTotal];
    tol = fin[kInnerFinTol];
  }
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] *= scale;
  double sk = 1.0, sp = 1.0, res = phibar, betan = 1.0;
  bool done = false;
  int k = 0;
  for (; k < kInnerSegment && !done; ++k) {
    double r[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const double w = twice >> e & 1 ? 2.0 : 1.0;
      const double vk = sk * v[e], y = d[e] * vk - beta * (sp * u[e]);
      r[0] += w * vk * y;
      r[1] += w * y * y;
      r[2] += w * vk * vk;
    }
    sums(r);
    // (as in inner_step_kernel)
    const double vp = r[0], pp = r[1], nv = r[2];
    const double alpha = nv > 0.0 ? vp / nv : 0.0;
    betan = sqrt(fmax(pp - alpha * vp, 0.0));
    const double eps = gs2 * beta, dbar = gc2 * beta;
    const double delta = gc1 * dbar + gs1 * alpha, gbar = -gs1 * dbar + gc1 * alpha;
    const double rho = hypot(gbar, betan);
    const double c = rho != 0.0 ? gbar / rho : 1.0, sn = rho != 0.0 ? betan / rho : 0.0;
    const double ib = betan != 0.0 ? 1.0 / betan : 0.0;
    const double sn1 = beta * ib != 0.0 ? beta * ib * sp : sk;
    const double ca = ib * (sk / sn1), cb = -alpha * ca;
    if (tid == 0) {
      cf[k][A] = ca;
      cf[k][B] = cb;
      cf[k][S] = sk;
      cf[k][DELTA] = delta;
      cf[k][EPS] = eps;
      cf[k][IR] = rho != 0.0 ? 1.0 / rho : 0.0;
      cf[k][PHI] = c * phibar;
    }
    phibar = -sn * phibar;
    res = fabs(phibar);
    total += 1.0;
    done = res <= tol || betan == 0.0 || total >= limit;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const double t = (d[e] * ca + cb) * v[e] - u[e];
      u[e] = v[e];
      v[e] = t;
    }
    beta = betan;
    sp = sk;
    sk = sn1;
    gc2 = gc1;
    gs2 = gs1;
    gc1 = c;
    gs1 = sn;
  }
  if (tid == 0) {
    st[kSBeta] = beta;
    st[kSC2] = gc2;
    st[kSS2] = gs2;
    st[kSC1] = gc1;
    st[kSS1] = gs1;
    st[kSPhiBar] = phibar;
    st[kSTotal] = total;
    fin[kInnerFinTol] = tol;
    fin[kInnerFinSteps] = total;
    fin[kInnerFinRes] = res;
    fin[kInnerFinBeta] = betan;
    // R y = phi, as in inner_finish_kernel
    double y1 = 0.0, y2 = 0.0, d1 = 0.0, e1 = 0.0, e2 = 0.0;
    for (int j = k - 1; j >= 0; --j) {
      const double y = (cf[j][PHI] - d1 * y1 - e2 * y2) * cf[j][IR];
      cf[j][Y] = cf[j][S] * y;
      y2 = y1;
      y1 = y;
      e2 = e1;
      e1 = cf[j][EPS];
      d1 = cf[j][DELTA];
    }
    g[0] = -d1 * y1 - e2 * y2;
    g[1] = -e1 * y1;
  }
  __syncthreads();
  constexpr int G = E < 8 ? E : 8;
#pragma unroll
  for (int e0 = 0; e0 < E; e0 += G) {
    double a[G], b[G], x[G];
#pragma unroll
    for (int e = 0; e < G; ++e) {
      const int q = min(tid + kRunThreads * (e0 + e), n - 1);
      a[e] = scale * v0[q];
      b[e] = first ? 0.0 : v1[q];
      x[e] = first ? 0.0 : xo[q] + g[0] * w1o[q] + g[1] * w2o[q];
    }
    for (int j = 0; j < k; ++j) {
      const double ca = cf[j][A], cb = cf[j][B], y = cf[j][Y];
#pragma unroll
      for (int e = 0; e < G; ++e) {
        x[e] += y * a[e];
        const double t = (d[e0 + e] * ca + cb) * a[e] - b[e];
        b[e] = a[e];
        a[e] = t;
      }
    }
    if (!done) {
      // another segment follows: the w recurrence itself, before v0 and v1 go
#pragma unroll 1
      for (int e = 0; e < G; ++e) {
        const int q = tid + kRunThreads * (e0 + e);
        if (q >= n) break;
        double dq = 0.0;
#pragma unroll
        for (int f = 0; f < G; ++f) dq = f == e ? d[e0 + f] : dq;
        double z = scale * v0[q], zp = first ? 0.0 : v1[q];
        double w1 = first ? 0.0 : w1o[q], w2 = first ? 0.0 : w2o[q];
        for (int j = 0; j < k; ++j) {
          const double w = (cf[j][S] * z - cf[j][DELTA] * w1 - cf[j][EPS] * w2) * cf[j][IR];
          w2 = w1;
          w1 = w;
          const double t = (dq * cf[j][A] + cf[j][B]) * z - zp;
          zp = z;
          z = t;
        }
        v0[q] = sk * z;
        v1[q] = sp * zp;
        w1o[q] = w1;
        w2o[q] = w2;
      }
    }
#pragma unroll
    for (int e = 0; e < G; ++e)
      if (tid + kRunThreads * (e0 + e) < n) xo[tid + kRunThreads * (e0 + e)] = x[e];
  }
}

// x_ij = x_ji^T for i > j of a full-layout vector's doubles, in place (through LDS).
__global__ __launch_bounds__(256) void inner_mirror_kernel(int o, int v, double* __restrict__ x2) {
  __shared__ double tile[kPackTile][kPackTile + 1];
  const int i = blockIdx.y / o, j = blockIdx.y % o;
  if (i <= j) return;
  const int64_t vv = (int64_t)v * v;
  double* __restrict__ out = x2 + (int64_t)blockIdx.y * vv;
  const double* __restrict__ src = x2 + (int64_t)(j * o + i) * vv;
  const int tid = threadIdx.x;
  const int nt = (v + kPackTile - 1) / kPackTile;
  const int tx = tid % kPackTile, ty = tid / kPackTile;
  for (int tl = blockIdx.x; tl < nt * nt; tl += gridDim.x) {
    const int a0 = (tl / nt) * kPackTile, b0 = (tl % nt) * kPackTile;
    __syncthreads();
    for (int r = ty; r < kPackTile; r += 256 / kPackTile) {  // tile[r][c] = x_ji[b0 + r][a0 + c]
      const int rr = b0 + r, cc = a0 + tx;
      tile[r][tx] = (rr < v && cc < v) ? src[(int64_t)rr * v + cc] : 0.0;
    }
    __syncthreads();
    for (int r = ty; r < kPackTile; r += 256 / kPackTile) {
      const int a = a0 + r, bb = b0 + tx;
      if (a < v && bb < v) out[(int64_t)a * v + bb] = tile[tx][r];
    }
  }
}

// ---- rotation of the occupied indices on the packed pair layout ----
//
// At one position e = (a, b) of the virtual grid a vector is the o x o matrix
// M^e_ij = x_ij^ab, whose lower triangle the packed layout keeps at the
// transposed position: M^e_ij = x_ji^ba for i > j. A workgroup takes 64
// positions closed under transposition, one per lane, and stages every packed
// pair at them in LDS.

// With nb odd, the blocks of the last row and column are the second half
// of a 2 x 2 group. When the v x v grid ends at most 4 elements into that
// last block (edge), the set of an off-diagonal block pair (Ta, nb - 1) is
// instead the 4 valid rows 8 (nb - 1) .. + 4 by the 8 columns of block Ta
// together with its transpose (all 64 positions in range, one set in place
// of two half-empty ones): at v = 180, 507 sets in place of 529, which two
// rounds of one workgroup per compute unit cover.
__host__ __device__ inline bool occ_set_edge(int v, int nb) { return (nb & 1) && v - 8 * (nb - 1) <= 4; }
__host__ __device__ inline int occ_set_count(int v, int nb) { return nb * nb - (occ_set_edge(v, nb) ? nb - 1 : 0); }

// Position set u (0 <= u < occ_set_count(v, nb)) over the 8 x 8 blocks of
// the v x v grid (nb = ceil(v / 8) per side): a diagonal block (T, T), or
// half h of an off-diagonal block pair (Ta < Tb): rows 8 Ta + 4 h .. + 4 by
// columns 8 Tb .. + 8 together with its transpose (the edge sets above
// aside). The blocks are taken in 2 x 2 groups (16 x 16 elements: two
// 128-byte lines of doubles per row), the upper group triangle row by row,
// so that the sets of a group, which share the lines they touch, run one
// after another on one XCD. A diagonal group holds 4 sets: (2g, 2g), (2g,
// 2g + 1) halves 0 and 1, (2g + 1, 2g + 1); an off-diagonal one 8: w = 4
// dTa + 2 dTb + h; with nb odd the last diagonal group holds 1 and the last
// column's groups 4 (dTb = 0; w = 2 dTa + h), or 2 edge sets (w = dTa).
__host__ __device__ inline bool occ_set_decode(int u, int nb, bool edge, bool* diag, int* a0, int* b0) {
  const int ng = (nb + 1) / 2;
  const bool odd = nb & 1;
  const int nhalf = edge ? 2 : 4;  // sets of a group in the last column (nb odd)
  for (int ga = 0; ga < ng; ++ga) {
    const int cd = odd && ga == ng - 1 ? 1 : 4, noff = ng - 1 - ga;
    const int row = cd + 8 * noff - (odd && noff > 0 ? 8 - nhalf : 0);
    if (u >= row) {
      u -= row;
      continue;
    }
    const int T = 2 * ga;
    if (u < cd) {
      *diag = u == 0 || u == 3;
      *a0 = *diag ? 8 * (T + (u == 3 ? 1 : 0)) : 8 * T + 4 * (u - 1);
      *b0 = *diag ? *a0 : 8 * (T + 1);
      return true;
    }
    u -= cd;
    const int gb = ga + 1 + u / 8, w = u % 8;
    const bool half = odd && gb == ng - 1;
    *diag = false;
    if (half && edge) {
      *a0 = 8 * (nb - 1);
      *b0 = 8 * (T + w);
      return true;
    }
    const int dTa = half ? w >> 1 : w >> 2, dTb = half ? 0 : (w >> 1) & 1, h = w & 1;
    *a0 = 8 * (T + dTa) + 4 * h;
    *b0 = 8 * (2 * gb + dTb);
    return true;
  }
  return false;  // u out of range
}

// Lane l's position (a, b) in the set, and the lane lT holding (b, a).
__host__ __device__ inline void occ_set_lane(bool diag, int l, int a0, int b0, int* a, int* b, int* lT) {
  if (diag) {
    const int r = l >> 3, c = l & 7;
    *a = a0 + r;
    *b = a0 + c;
    *lT = 8 * c + r;
  } else if (l < 32) {
    const int r = l >> 3, c = l & 7;
    *a = a0 + r;
    *b = b0 + c;
    *lT = 32 + 4 * c + r;
  } else {
    const int m = l - 32, r = m >> 2, c = m & 3;
    *a = b0 + r;
    *b = a0 + c;
    *lT = 8 * c + r;
  }
}

constexpr int kOccMax = 24;  // 64 positions of o (o + 1) / 2 pairs fit a workgroup's LDS (154 KB at 24)

struct OccArgs {
  int o, v, nb, units, dwg;  // dwg: units rounded up to a multiple of 8; then workgroups of singles
  const double* rot;         // row j: coefficients of the rotated index j
  VecIn src;
  VecOut dst;
  double rs;
  double* parts;
};

// IN: src is a full-layout b, dst the packed D^1/2 R sym(b) R^T, with the shares
// of ||sym(b)||^2 and ||D^1/2 sym(b)||^2 (parts[g], parts[G + g]). Otherwise src
// is a packed x and dst the full layout of D^1/2 R x R^T, both halves. R acts on
// the occupied indices. One wave per two columns j of the rotated matrix: it
// forms t_kj = sum_l M_kl R_jl for all k in registers (KMAX >= o of them), then
// Y_ij = sum_k R_ik t_kj for i <= j. Bound by memory (o = 20, v = 180: 104 MB and
// 56 MB), the sums of one workgroup per CU not overlapping its loads: in 122 us,
// out 107; as two products over the full layout and a packing pass, 158 and 176.
template <int KMAX, bool IN>
__global__ __launch_bounds__(32 * KMAX < 64 ? 64 : 32 * KMAX) void inner_occ_kernel(OccArgs p) {
  extern __shared__ __attribute__((aligned(16))) double M[];  // [pair][64]
  __shared__ double red[2][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = blockDim.x >> 6;
  const int o = p.o, v = p.v, npair = o * (o + 1) / 2;
  const int64_t vv = (int64_t)v * v;
  const int ov = o * v;
  double s_plain = 0.0, s_scaled = 0.0;
  auto row_of = [&](int k) { return k * o - k * (k - 1) / 2 - k; };  // P(k, l) = row_of(k) + l, k <= l
  if ((int)blockIdx.x >= p.dwg) {
    const int q = (blockIdx.x - p.dwg) * blockDim.x + tid;
    if (q < ov) {
      const int j = q / v, a = q - j * v;
      double y = 0.0;
      for (int l = 0; l < o; ++l) y += p.rot[j * o + l] * p.src.x1[l * v + a];
      p.dst.x1[q] = p.rs * y;
      const double x = p.src.x1[q];
      s_plain = x * x;
      s_scaled = (p.rs * x) * (p.rs * x);
    }
  } else {
    // each XCD takes a contiguous range of sets (neighbours share lines)
    const int u = (int)(blockIdx.x & 7) * (p.dwg >> 3) + (int)(blockIdx.x >> 3);
    bool diag = false;
    int a0 = 0, b0 = 0;
    if (u < p.units && occ_set_decode(u, p.nb, occ_set_edge(v, p.nb), &diag, &a0, &b0)) {
      int a, b, lt;
      occ_set_lane(diag, lane, a0, b0, &a, &b, &lt);
      const bool in = a < v && b < v;
      const int64_t e = in ? (int64_t)a * v + b : 0, et = in ? (int64_t)b * v + a : 0;
      // stage: four pairs' loads in flight per wave
      int k = 0, l = wave;  // pair (k, l), k <= l
      for (; k < o && l >= o; ++k) l -= o - k - 1;
      for (int P = wave; P < npair; P += 4 * nw) {
        double x[4], w[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          x[c] = w[c] = 0.0;
          if (P + c * nw < npair) {
            if constexpr (IN) {
              const double m = p.src.x2[(int64_t)(k * o + l) * vv + e], mt = p.src.x2[(int64_t)(l * o + k) * vv + et];
              x[c] = 0.5 * (m + mt);
              w[c] = k == l ? 1.0 : 2.0;
            } else {
              x[c] = p.src.x2[(int64_t)(P + c * nw) * vv + e];
            }
          }
          l += nw;
          for (; k < o && l >= o; ++k) l -= o - k - 1;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (P + c * nw < npair) {
            M[(P + c * nw) * 64 + lane] = in ? x[c] : 0.0;
            if (IN && in) {
              s_plain += w[c] * x[c] * x[c];
              s_scaled += w[c] * x[c] * x[c];
            }
          }
      }
      __syncthreads();
      const double* xl = M + lane;
      const double* xt = M + lt;
      for (int j0 = 2 * wave; j0 < o; j0 += 2 * nw) {
        const int j1 = min(j0 + 1, o - 1);
        double t[KMAX][2];
#pragma unroll
        for (int kk = 0; kk < KMAX; ++kk) t[kk][0] = t[kk][1] = 0.0;
        for (int ll = 0; ll < o; ++ll) {
          const double u0 = p.rot[j0 * o + ll], u1 = p.rot[j1 * o + ll];
          const int rl = row_of(ll);
#pragma unroll
          for (int kk = 0; kk < KMAX; ++kk) {
            const int kc = min(kk, o - 1);  // (rows past o: never used)
            const double m = kc <= ll ? xl[(row_of(kc) + ll) * 64] : xt[(rl + kc) * 64];
            t[kk][0] += m * u0;
            t[kk][1] += m * u1;
          }
        }
        for (int i = 0; i <= j1; ++i) {
          double y0 = 0.0, y1 = 0.0;
#pragma unroll
          for (int kk = 0; kk < KMAX; ++kk) {
            const double c = kk < o ? p.rot[i * o + kk] : 0.0;
            y0 += c * t[kk][0];
            y1 += c * t[kk][1];
          }
          if (!in) continue;
          if constexpr (IN) {
            double* out = p.dst.x2 + e;
            if (i <= j0) out[(int64_t)(row_of(i) + j0) * vv] = y0;
            if (j1 > j0) out[(int64_t)(row_of(i) + j1) * vv] = y1;
          } else {
            double *out = p.dst.x2 + e, *outt = p.dst.x2 + et;
            if (i <= j0) out[(int64_t)(i * o + j0) * vv] = y0;
            if (i < j0) outt[(int64_t)(j0 * o + i) * vv] = y0;
            if (j1 > j0) {
              out[(int64_t)(i * o + j1) * vv] = y1;
              if (i < j1) outt[(int64_t)(j1 * o + i) * vv] = y1;
            }
          }
        }
      }
    }
  }
  if constexpr (IN) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
      s_plain += __shfl_xor(s_plain, m, 64);
      s_scaled += __shfl_xor(s_scaled, m, 64);
    }
    if (lane == 0) {
      red[0][wave] = s_plain;
      red[1][wave] = s_scaled;
    }
    __syncthreads();
    if (tid == 0) {
      double r0 = 0.0, r1 = 0.0;
      for (int q = 0; q < nw; ++q) {
        r0 += red[0][q];
        r1 += red[1][q];
      }
      p.parts[blockIdx.x] = r0;
      p.parts[gridDim.x + blockIdx.x] = r1;
    }
  }
}

template <int KMAX, bool IN>
void launch_occ(const OccArgs& p, unsigned grid, hipStream_t s) {
  const size_t lds = (size_t)p.o * (p.o + 1) / 2 * 64 * sizeof(double);
  if (lds > 48 * 1024)
    PNK_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&inner_occ_kernel<KMAX, IN>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  inner_occ_kernel<KMAX, IN><<<grid, 64 * ((p.o + 1) / 2), lds, s>>>(p);
  PNK_CHECK_LAUNCH();
}
template <bool IN>
int occ_rotation(const FockEigen& e, VecIn src, VecOut dst, double rs, double* parts, hipStream_t s) {
  OccArgs p;
  p.o = e.o; p.v = e.v;
  p.nb = (e.v + 7) / 8;
  p.units = occ_set_count(e.v, p.nb);
  p.dwg = (p.units + 7) / 8 * 8;
  p.rot = IN ? e.ut_o : e.u_o;
  p.src = src; p.dst = dst; p.rs = rs; p.parts = parts;
  const int threads = 64 * ((e.o + 1) / 2);
  const unsigned grid = (unsigned)(p.dwg + ceil_div((int64_t)e.o * e.v, threads));
  switch ((e.o + 3) / 4) {
    case 1: launch_occ<4, IN>(p, grid, s); break;
    case 2: launch_occ<8, IN>(p, grid, s); break;
    case 3: launch_occ<12, IN>(p, grid, s); break;
    case 4: launch_occ<16, IN>(p, grid, s); break;
    case 5: launch_occ<20, IN>(p, grid, s); break;
    default: launch_occ<24, IN>(p, grid, s); break;
  }
  return (int)grid;
}

int pair_rows(const InnerSolve& q) { return std::min(q.eig.o * (q.eig.o + 1) / 2 + 1, kInnerMaxRows); }
int full_groups(const InnerSolve& q) { return (int)std::min<int64_t>(ceil_div(q.n, 256), 1024); }
int npair(const InnerSolve& q) { return q.packed ? q.eig.o * (q.eig.o + 1) / 2 : q.eig.o * q.eig.o; }

Args args_of(const InnerSolve& q, int parity, double singles_scale) {
  Args p;
  p.o = q.eig.o; p.v = q.eig.v;
  p.blocks = q.blocks; p.npair = npair(q); p.segs = q.segs;
  p.parity = parity;
  p.eps_o = q.eig.eps_o; p.eps_v = q.eig.eps_v;
  p.v0 = q.v0; p.v1 = q.v1;
  p.part_in = q.parts + parity * 3 * kInnerMaxParts;
  p.part_out = q.parts + (1 - parity) * 3 * kInnerMaxParts;
  p.coef = q.coef;
  p.state = q.state;
  p.sscale = singles_scale;
  return p;
}

GemmDesc product(int M, int N, int K, int64_t am, int64_t ak, int64_t bk, int64_t bn, int64_t cm) {
  GemmDesc d;
  d.M = M; d.N = N; d.K = K;
  d.a_m = am; d.a_k = ak; d.b_k = bk; d.b_n = bn; d.c_m = cm; d.c_n = 1;
  return d;
}

// The occupied indices of a full-layout vector, through tmp.
// forward: y[i'] = sum_i U[i][i'] x[i], U[i][i'] = ut[i' o + i]
void rotate_occ(const FockEigen& e, bool forward, VecIn in, double* tmp, VecOut out, hipStream_t s) {
  const int o = e.o, v = e.v;
  const int64_t vv = (int64_t)v * v, am = forward ? o : 1, ak = forward ? 1 : o;
  gemm64(product(o, v, o, am, ak, v, 1, v), e.ut_o, in.x1, out.x1, s);
  GemmDesc d = product(o, (int)(o * vv), o, am, ak, o * vv, 1, o * vv);
  gemm64(d, e.ut_o, in.x2, tmp, s);
  d = product(o, (int)vv, o, am, ak, vv, 1, vv);
  d.nb0 = o; d.b_b0 = o * vv; d.c_b0 = o * vv;
  gemm64(d, e.ut_o, tmp, out.x2, s);
}

}  // namespace

void inner_shape(InnerSolve& q, bool packed) {
  const int64_t o = q.eig.o, vv = (int64_t)q.eig.v * q.eig.v;
  q.packed = packed;
  const int64_t np = npair(q);
  q.n = o * q.eig.v + np * vv;
  // About 900 workgroups of at least 1024 elements: every one adds all
  // shares of the launch before, and three or four fit a CU (o = 20, v = 180:
  // 211 rows x 4; o = 10, v = 90: 56 x 8)
  q.blocks = (int)std::min<int64_t>(np + 1, kInnerMaxRows);
  q.segs = (int)std::max<int64_t>(1, std::min<int64_t>(ceil_div(vv, 1024), 900 / q.blocks));
}

// (the sets' workgroups write at most ceil(v / 8)^2 + 8 + o v / 64 shares)
bool occ_sets_apply(const InnerSolve& q) {
  const int64_t nb = (q.eig.v + 7) / 8;
  return q.packed && q.eig.o <= kOccMax && nb * nb + 8 + q.eig.v <= 16 * kInnerMaxRows;
}

int inner_load(const InnerSolve& q, VecIn b, double* tmp1, double* tmp2, double singles_scale, hipStream_t s) {
  const double rs = std::sqrt(singles_scale);
  const int64_t ov = (int64_t)q.eig.o * q.eig.v;
  if (q.eig.ut_o) {
    if (occ_sets_apply(q)) return occ_rotation<true>(q.eig, b, {q.v0, q.v0 + ov}, rs, q.norm_parts, s);
    rotate_occ(q.eig, true, b, tmp1, {tmp2, tmp2 + ov}, s);
    b = {tmp2, tmp2 + ov};
  }
  int np;
  if (q.packed) {
    np = kPackBlocksX * pair_rows(q);
    inner_pack<<<dim3(kPackBlocksX, pair_rows(q)), 256, 0, s>>>(q.eig.o, q.eig.v, b, rs, q.v0, q.norm_parts);
  } else {
    np = full_groups(q);
    inner_copy_in<<<np, 256, 0, s>>>(q.n, ov, b, rs, q.v0, q.norm_parts);
  }
  PNK_CHECK_LAUNCH();
  return np;
}

void inner_begin(const InnerSolve& q, int nshares, double rtol, int limit, hipStream_t s) {
  inner_begin_kernel<<<1, 256, 0, s>>>(q.norm_parts, nshares, q.state, rtol, (double)limit);
  PNK_CHECK_LAUNCH();
}

namespace {
template <bool PACKED>
void launch_step(const InnerSolve& q, const Args& p, hipStream_t s) {
  const dim3 grid(q.segs, q.blocks);
  const size_t lds = q.eig.v * sizeof(double);
  // eight elements per thread where a workgroup has more than 1024
  if (ceil_div((int64_t)q.eig.v * q.eig.v, q.segs) > 1024) inner_step_kernel<PACKED, 8><<<grid, 256, lds, s>>>(p);
  else inner_step_kernel<PACKED, 4><<<grid, 256, lds, s>>>(p);
}
}  // namespace

// Up to 16 elements a thread: with 24 the registers spill (4.4 us a step in
// place of 2.6 at 16; a launch for each step takes 6.1 at any such length).
bool inner_runs_whole(const InnerSolve& q) { return q.n <= 16 * kRunThreads; }

namespace {
template <bool PACKED>
void launch_run(const InnerSolve& q, const Args& p, bool first, int nshares, double rtol, double limit, hipStream_t s) {
  const int n = (int)q.n;
  auto go = [&](auto kernel) {
    kernel<<<1, kRunThreads, 0, s>>>(p, n, first, q.norm_parts, nshares, rtol, limit, q.v0, q.v1, q.w1, q.w2, q.x);
  };
  if (n <= 2 * kRunThreads) go(inner_run_kernel<PACKED, 2>);
  else if (n <= 8 * kRunThreads) go(inner_run_kernel<PACKED, 8>);
  else go(inner_run_kernel<PACKED, 16>);
}
}  // namespace

void inner_run(const InnerSolve& q, bool first, int nshares, double rtol, int limit, double singles_scale, hipStream_t s) {
  const Args p = args_of(q, 0, singles_scale);
  if (q.packed) launch_run<true>(q, p, first, nshares, rtol, limit, s);
  else launch_run<false>(q, p, first, nshares, rtol, limit, s);
  PNK_CHECK_LAUNCH();
}

void inner_step(const InnerSolve& q, int parity, double singles_scale, hipStream_t s) {
  const Args p = args_of(q, parity, singles_scale);
  if (q.packed) launch_step<true>(q, p, s);
  else launch_step<false>(q, p, s);
  PNK_CHECK_LAUNCH();
}

bool inner_is_step_kernel(const void* func) {
  return func == reinterpret_cast<const void*>(&inner_step_kernel<true, 4>) ||
         func == reinterpret_cast<const void*>(&inner_step_kernel<true, 8>) ||
         func == reinterpret_cast<const void*>(&inner_step_kernel<false, 4>) ||
         func == reinterpret_cast<const void*>(&inner_step_kernel<false, 8>);
}

void inner_finish(const InnerSolve& q, int steps, bool first_segment, bool rebase, int parity, double singles_scale,
                  hipStream_t s) {
  const Args p = args_of(q, parity, singles_scale);
  const int64_t vv = (int64_t)q.eig.v * q.eig.v;
  const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(vv, 1024), 2048 / q.blocks)), q.blocks);
  const size_t lds = q.eig.v * sizeof(double);
  if (rebase) {
    if (q.packed) inner_rebase_kernel<true><<<grid, 256, lds, s>>>(p, steps, q.v0, q.v1, q.w1, q.w2, q.x, first_segment);
    else inner_rebase_kernel<false><<<grid, 256, lds, s>>>(p, steps, q.v0, q.v1, q.w1, q.w2, q.x, first_segment);
    inner_rebase_state<<<1, 64, 0, s>>>(q.state + parity * kInnerState);
  } else if (q.packed) {
    inner_finish_kernel<true><<<grid, 256, lds, s>>>(p, steps, q.w1, q.w2, q.x, first_segment);
  } else {
    inner_finish_kernel<false><<<grid, 256, lds, s>>>(p, steps, q.w1, q.w2, q.x, first_segment);
  }
  PNK_CHECK_LAUNCH();
}

void inner_unload(const InnerSolve& q, double* tmp1, double* tmp2, double singles_scale, VecOut out, hipStream_t s) {
  const double rs = std::sqrt(singles_scale);
  const int o = q.eig.o, v = q.eig.v;
  const int64_t ov = (int64_t)o * v;
  if (q.eig.ut_o && occ_sets_apply(q)) {
    occ_rotation<false>(q.eig, {q.x, q.x + ov}, out, rs, nullptr, s);
    return;
  }
  const VecOut full = q.eig.ut_o ? VecOut{tmp1, tmp1 + ov} : out;
  if (q.packed) inner_unpack<<<dim3(kPackBlocksX, o * o + 1), 256, 0, s>>>(o, v, q.x, rs, full);
  else inner_copy_out<<<full_groups(q), 256, 0, s>>>(q.n, ov, q.x, rs, full);
  PNK_CHECK_LAUNCH();
  if (q.eig.ut_o) {
    rotate_occ(q.eig, false, {full.x1, full.x2}, tmp2, out, s);
    if (q.packed) {
      inner_mirror_kernel<<<dim3(kPackBlocksX, o * o), 256, 0, s>>>(o, v, out.x2);
      PNK_CHECK_LAUNCH();
    }
  }
}

// forward: y[a'][b'] = sum U[a][a'] x[a][b] U[b][b'], U[a][a'] = ut[a' v + a]
void inner_rotate_vir(const FockEigen& e, bool forward, int64_t rows, double* x, double* tmp, hipStream_t s) {
  const int o = e.o, v = e.v;
  const int64_t vv = (int64_t)v * v, ov = (int64_t)o * v;
  // the second index of the singles and of every block: rows of length v
  const int64_t bk = forward ? 1 : v, bn = forward ? v : 1;
  gemm64(product((int)(o + rows * v), v, v, v, 1, bk, bn, v), x, e.ut_v, tmp, s);
  GemmDesc d = product(v, v, v, forward ? v : 1, forward ? 1 : v, v, 1, v);
  d.nb0 = (int)rows; d.b_b0 = vv; d.c_b0 = vv;
  gemm64(d, e.ut_v, tmp + ov, x + ov, s);
  PNK_HIP(hipMemcpyAsync(x, tmp, ov * sizeof(double), hipMemcpyDeviceToDevice, s));
}

int inner_set_positions(int v, int* a, int* b, int* lt, int64_t cap) {
  if (v < 1 || !a || !b || !lt) return -1;
  const int nb = (v + 7) / 8, n = occ_set_count(v, nb);
  if ((int64_t)n * 64 > cap) return -1;
  const bool edge = occ_set_edge(v, nb);
  for (int u = 0; u < n; ++u) {
    bool diag = false;
    int a0 = 0, b0 = 0;
    if (!occ_set_decode(u, nb, edge, &diag, &a0, &b0)) return -1;
    for (int l = 0; l < 64; ++l) occ_set_lane(diag, l, a0, b0, &a[u * 64 + l], &b[u * 64 + l], &lt[u * 64 + l]);
  }
  return n;
}

}  // namespace pnk
