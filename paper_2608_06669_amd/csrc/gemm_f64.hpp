// FP64 matrix-core product with direct-to-LDS panels (see gemm.hpp for the
// operand addressing). Included by gemm.hip only.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace pnk {
namespace f64pipe {

typedef double d2 __attribute__((ext_vector_type(2)));

struct Args {
  int M, N, K, nb0;
  int bm, bn;      // tile
  int tm, tn;      // tiles along M and N
  int nfull;       // tiles computed in one piece: C written directly
  int ntail, ts;   // the other tiles, each cut into ts chunks of kchunk along K
  int kchunk;      // (a multiple of the panel depth)
  const double *A, *B, *A2, *B2;  // A2, B2: optional second product into the same sum
  int64_t lda, a_b0, a_b1;
  int64_t ldb, b_b0, b_b1;
  double* C;
  const double* Cin;  // C = alpha sum + beta Cin, at C's strides
  int64_t c_m, c_n, c_b0, c_b1;
  double alpha, beta;
  double* ws;      // chunk sums [chunk][tail tile][wr * wc]
  int wr, wc;      // rows and columns a tile's sums keep (the tile's, or fewer if the matrix has fewer)
};

// Tile t of the product: batch entry, then groups of up to 8 row tiles with
// the row tile fastest, so workgroups that run together share A and B panels
// in their XCD's L2.
__device__ inline void tile_coords(const Args& p, int t, int* b, int* im, int* in) {
  constexpr int kGroupM = 8;
  const int per = p.tm * p.tn;
  *b = t / per;
  t -= *b * per;
  const int gsize = kGroupM * p.tn;
  const int grp = t / gsize, first = grp * kGroupM;
  const int gm = min(p.tm - first, kGroupM);
  const int rem = t - grp * gsize;
  *im = first + rem % gm;
  *in = rem / gm;
}

// XCD x receives block ids x, x + 8, ...: give it the contiguous range of
// q + (x < r) items that starts at x q + min(x, r)
__device__ inline int xcd_range(int e, int n) {
  const int q = n >> 3, r = n & 7, x = e & 7;
  return x * q + min(x, r) + (e >> 3);
}

template <int N>
__device__ inline void wait_vm_lgkm0() {  // vmcnt(N), lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

// One direct-to-LDS load per lane, 16 or 4 bytes; lane l's bytes land at dst
// + l times their number.
template <bool VEC>
__device__ inline void to_lds(const void* src, uint32_t* dst) {
  if constexpr (VEC) __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
  else __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)dst, 4, 0, 0);
}

// A launch holds fewer than 2^32 threads along x: products of more tiles and
// chunks than this take gridDim.y rows of them (a multiple of 8, as
// xcd_range needs).
constexpr int64_t kMaxGridX = int64_t(1) << 23;

// 16 zero bytes that a remainder panel reads in place of k past the end
static __device__ __align__(16) double zero_src[2];

// One workgroup of 4 waves (2 x 2) forms a BM x BN tile with the 4x4x4 f64
// instruction. 8-deep panels of A and B go straight from global memory into
// a ring of four LDS stages (three panels in flight while the fourth is
// multiplied). A_KC, B_KC: the operand is contiguous along k (else along its
// row index m or n). VEC: its rows are 16-byte aligned and two elements at a
// time are whole (16 bytes per lane and load); otherwise 4 bytes per lane, so
// rows of any alignment and length take the same path.
// Operands are read from LDS 16 bytes at a time: two consecutive k of a row
// (k-contiguous panels, stored [row][8] with the four 16-byte chunks of a row
// at slot chunk ^ ((row / 4) % 4), rows counted within the wave's half) or two
// consecutive rows at one k (stored [k][rows]). Lanes 16 g .. 16 g + 15 take k = 2 g and 2 g + 1 of a panel, one
// for each of its two instruction steps. The fragments of a panel are read
// while the panel before it is multiplied, so neither the LDS latency nor the
// barrier is on the matrix cores' path.
// Limits (MI355X, operands with full mantissas): the 4x4x4 instruction alone,
// operands in registers, sustains 72 TFLOP/s. In a residual at o = 20, v = 180
// the matrix pipes are busy for 88 to 92 % of the cycles with 64 x 128 tiles, 80
// with 64 x 64, 75 with 72 x 64 and 71 where both operands are contiguous along
// their rows (LDS bank conflicts in 44 % of its cycles), at a clock of 2.0 to 2.3
// GHz where the streaming kernels beside them get 2.5. 3600^3 runs at 62-65 TFLOP/s (the former
// kernel, 16-deep panels in three stages with the fragments read after the
// barrier, 1640-1710 us in place of 1441-1492), 1183^3 with rows of odd length,
// which it could not take, at 37-41 (4-byte loads).
// Tiles of 48, 72 or 80 rows serve row counts that multiples of 64 fit badly
// (the pair rows of the ladders): 136 x 12880 x 10440 takes 990 us with 72 rows
// where 64 took 1430, 78 x 5360 x 4096 118 with 80 (142), 20 x 180 x 108000 126
// with 48 (165); 210 x 20104 x 16296 2740 with 72 (2860 with 64 x 128).
// A contraction that is not whole panels starts with its remainder, zeros in
// place of the missing k, in the prologue: the loop sees whole panels only.
//
// ASC: each matrix instruction takes four consecutive k, so that sums run in
// ascending k. It costs nothing where both operands are contiguous along their
// rows; along k, one 16-byte read per fragment becomes two of 8 bytes (all
// products of a residual that way: 14.5 in place of 13.6 ms at o = 20, v =
// 180), so those kernels otherwise take k = 0, 2, 4, 6 and 1, 3, 5, 7.
//
// LONG: rows of any length and direction, the lanes' offsets in 64 bits. In 32
// bits, half the registers, they reach 128 rows of up to 2^22 elements.
template <int BM, int BN, bool A_KC, bool B_KC, bool VEC, bool LONG = false, bool ASC = !A_KC && !B_KC>
__global__ __launch_bounds__(256, 2) void gemm_f64_pipe(Args p) {
  constexpr int BK = 8, NT = 256, AE = BM * BK, BE = BN * BK, SE = AE + BE;
  constexpr int WTM = BM / 2, WTN = BN / 2, TMI = WTM / 4, TNI = WTN / 16;
  constexpr int EPL = VEC ? 4 : 1;                                // dwords per lane and load
  // loads per thread and panel; where A's are not whole ones, every wave takes
  // the last with its first RA lanes (all waves count the same loads)
  constexpr int FA = AE * 2 / (EPL * NT), RA = (AE * 2 / EPL - FA * NT) / 4, CA = FA + (RA > 0), CB = BE * 2 / (EPL * NT);
  static_assert((FA * NT + 4 * RA) * EPL == AE * 2 && CB >= 1 && CB * EPL * NT == BE * 2, "whole loads");
  static_assert((A_KC || TMI % 2 == 0) && (B_KC || TNI % 2 == 0), "row pairs");
  __shared__ __attribute__((aligned(1024))) double st0[SE], st1[SE], st2[SE], st3[SE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // (a grid of several rows has this width; its last one may pass the end)
  const uint32_t item = blockIdx.y * (uint32_t)kMaxGridX + blockIdx.x;
  if (item >= (uint32_t)(p.nfull + p.ntail * p.ts)) return;
  int tile, split = 0, nsplit = 1;
  if ((int)item < p.nfull) {
    tile = xcd_range(item, p.nfull);
  } else {
    nsplit = p.ts;
    const int e = xcd_range(item - p.nfull, p.ntail * p.ts);
    split = e / p.ntail;
    tile = p.nfull + e - split * p.ntail;
  }
  int b, im, in;
  tile_coords(p, tile, &b, &im, &in);
  const int b0 = b % p.nb0, b1 = b / p.nb0;
  const int m0 = im * BM, n0 = in * BN;
  const int kbeg = nsplit > 1 ? split * p.kchunk : 0;
  const int klen = (nsplit > 1 ? min(p.K, kbeg + p.kchunk) : p.K) - kbeg;
  const bool dual = p.A2 != nullptr;
  const int nf = klen / BK, rem = klen - nf * BK;   // whole panels of one product, columns of its remainder
  const int np = rem ? (dual ? 2 : 1) : 0;          // remainder panels, taken first
  const int nk = np + (dual ? 2 * nf : nf);

  // this thread's loads j NT + tid: byte offsets from the tile's corner
  // (rows past the matrix read its last ones, whose outputs are not written)
  // and the k they hold
  using Offset = std::conditional_t<LONG, int64_t, uint32_t>;
  Offset oa[CA], ob[CB];
  auto place = [&](int j, bool part, bool kc, int rows, int left, int64_t ld, Offset* off, int* k) {
    const int w = (j * NT + (part ? wave * RA + min(lane, RA - 1) : tid)) * EPL;  // dword of the panel
    const int c = w >> 2, half = (w >> 1) & 1;  // 16-byte chunk, element of it
    int r, kk;
    if (kc) {
      r = c >> 2;
      kk = 2 * ((c & 3) ^ ((r % (rows / 2) >> 2) & 3)) + half;
      r = min(r, left - 1);
      *off = (Offset)(((int64_t)r * ld + kk) * 8 + (w & 1) * 4);
    } else {
      kk = c / (rows / 2);
      r = min(2 * (c % (rows / 2)) + half, VEC ? left - 2 : left - 1);
      *off = (Offset)(((int64_t)kk * ld + r) * 8 + (w & 1) * 4);
    }
    *k = kk;
  };
  const char* A1 = (const char*)(p.A + b0 * p.a_b0 + b1 * p.a_b1 + (A_KC ? m0 * p.lda + kbeg : kbeg * p.lda + m0));
  const char* B1 = (const char*)(p.B + b0 * p.b_b0 + b1 * p.b_b1 + (B_KC ? n0 * p.ldb + kbeg : kbeg * p.ldb + n0));
  const char* A2 = dual ? A1 + ((const char*)p.A2 - (const char*)p.A) : A1;
  const char* B2 = dual ? B1 + ((const char*)p.B2 - (const char*)p.B) : B1;
  const int64_t sa = A_KC ? 8 : 8 * p.lda, sb = B_KC ? 8 : 8 * p.ldb;  // bytes from one k to the next
  int kq;
#pragma unroll
  for (int j = 0; j < CA; ++j) place(j, j == FA, A_KC, BM, p.M - m0, p.lda, &oa[j], &kq);
#pragma unroll
  for (int j = 0; j < CB; ++j) place(j, false, B_KC, BN, p.N - n0, p.ldb, &ob[j], &kq);

  auto load_a = [&](int j, const char* src, double* st) {
    if (j < FA) to_lds<VEC>(src, (uint32_t*)st + (j * NT + wave * 64) * EPL);
    else if (lane < RA) to_lds<VEC>(src, (uint32_t*)st + (j * NT + wave * RA) * EPL);
  };
  // whole panel f of the first (f < nf) or second product; past the last
  // one, the last again (never read)
  auto issue = [&](double* st, int t) {
    int f = min(t - np, nk - np - 1);
    const bool second = f >= nf;
    f -= second ? nf : 0;
    const char* a = (second ? A2 : A1) + (rem + (int64_t)f * BK) * sa;
    const char* bq = (second ? B2 : B1) + (rem + (int64_t)f * BK) * sb;
    // (kept in scalar registers: folded into the lanes' offsets, the loop
    // would add 64-bit vectors for every load)
    asm volatile("" : "+s"(a), "+s"(bq));
#pragma unroll
    for (int j = 0; j < CA; ++j) load_a(j, a + oa[j], st);
#pragma unroll
    for (int j = 0; j < CB; ++j) to_lds<VEC>(bq + ob[j], (uint32_t*)(st + AE) + (j * NT + wave * 64) * EPL);
  };
  // remainder panel t (product t): k = 0 .. rem - 1
  auto issue_rem = [&](double* st, int t) {
    const char *a = t ? A2 : A1, *bq = t ? B2 : B1, *z = (const char*)zero_src;
#pragma unroll
    for (int j = 0; j < CA; ++j) {
      Offset o;
      int k;
      place(j, j == FA, A_KC, BM, p.M - m0, p.lda, &o, &k);
      load_a(j, k < rem ? a + o : z, st);
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      Offset o;
      int k;
      place(j, false, B_KC, BN, p.N - n0, p.ldb, &o, &k);
      to_lds<VEC>(k < rem ? bq + o : z, (uint32_t*)(st + AE) + (j * NT + wave * 64) * EPL);
    }
  };
  auto issue_first = [&](double* st, int t) {
    if (t < np) issue_rem(st, t);
    else if (nk > np) issue(st, t);
    else issue_rem(st, np - 1);  // remainder panels only: again the last (never read)
  };

  double acc[TMI][TNI];
#pragma unroll
  for (int i = 0; i < TMI; ++i)
#pragma unroll
    for (int j = 0; j < TNI; ++j) acc[i][j] = 0.0;
  struct Frag {
    double a[2][TMI], b[2][TNI];
  };
  const int g = lane >> 4;
  auto kr = [&](int e) { return ASC ? 4 * e + g : 2 * g + e; };  // k of this lane's e-th operand
  auto read = [&](Frag& f, const double* st) {
    if constexpr (A_KC) {
#pragma unroll
      for (int i = 0; i < TMI; ++i) {
        const int m = wm * WTM + i * 4 + (lane & 3);
        if constexpr (ASC) {
#pragma unroll
          for (int e = 0; e < 2; ++e) f.a[e][i] = st[m * BK + 2 * ((2 * e + (g >> 1)) ^ (i & 3)) + (g & 1)];
        } else {
          const d2 x = *reinterpret_cast<const d2*>(st + m * BK + 2 * (g ^ (i & 3)));
          f.a[0][i] = x[0];
          f.a[1][i] = x[1];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int i = 0; i < TMI; i += 2) {
          const d2 x = *reinterpret_cast<const d2*>(st + kr(e) * BM + wm * WTM + i * 4 + 2 * (lane & 3));
          f.a[e][i] = x[0];
          f.a[e][i + 1] = x[1];
        }
    }
    if constexpr (B_KC) {
#pragma unroll
      for (int j = 0; j < TNI; ++j) {
        const int n = wn * WTN + j * 16 + (lane & 15);
        if constexpr (ASC) {
#pragma unroll
          for (int e = 0; e < 2; ++e)
            f.b[e][j] = st[AE + n * BK + 2 * ((2 * e + (g >> 1)) ^ ((n >> 2) & 3)) + (g & 1)];
        } else {
          const d2 x = *reinterpret_cast<const d2*>(st + AE + n * BK + 2 * (g ^ ((n >> 2) & 3)));
          f.b[0][j] = x[0];
          f.b[1][j] = x[1];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int j = 0; j < TNI; j += 2) {
          const d2 x = *reinterpret_cast<const d2*>(st + AE + kr(e) * BN + wn * WTN + j * 16 + 2 * (lane & 15));
          f.b[e][j] = x[0];
          f.b[e][j + 1] = x[1];
        }
    }
  };
  auto multiply = [&](const Frag& f) {
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < TMI; ++i)
#pragma unroll
        for (int j = 0; j < TNI; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(f.a[e][i], f.b[e][j], acc[i][j], 0, 0, 0);
  };
  Frag fr;
  // step t: panel t + 1 has landed (panel t + 2's loads may be in flight) and
  // every wave is past its reads of panel t - 1's stage; refill that stage
  // with panel t + 3, read panel t + 1's fragments and multiply panel t's.
  // (A plain barrier: the workgroup fence of __syncthreads would wait for all
  // loads in flight.)
  auto step = [&](int t, const double* next, double* fill) {
    wait_vm_lgkm0<CA + CB>();
    __builtin_amdgcn_s_barrier();
    issue(fill, t + 3);
    Frag fn;
    read(fn, next);
    multiply(fr);
    fr = fn;
  };
  issue_first(st0, 0);
  issue_first(st1, 1);
  issue_first(st2, 2);
  wait_vm_lgkm0<2 * (CA + CB)>();
  __builtin_amdgcn_s_barrier();
  read(fr, st0);
  // whole rounds of four in the loop, the rest after it (steps under a
  // condition in the loop would make the compiler wait for every load)
  int t = 0;
  for (; t + 4 < nk; t += 4) {
    step(t, st1, st3);
    step(t + 1, st2, st0);
    step(t + 2, st3, st1);
    step(t + 3, st0, st2);
  }
  // 1 to 4 panels left, the first one's fragments read already; the fourth
  // has yet to be loaded, into the stage read before the last barrier's step
  wait_vm_lgkm0<0>();
  if (t + 3 < nk) {
    __builtin_amdgcn_s_barrier();
    issue(st3, t + 3);
    wait_vm_lgkm0<0>();
  }
  __builtin_amdgcn_s_barrier();
  multiply(fr);
  if (t + 1 < nk) { read(fr, st1); multiply(fr); }
  if (t + 2 < nk) { read(fr, st2); multiply(fr); }
  if (t + 3 < nk) { read(fr, st3); multiply(fr); }

  auto row_of = [&](int i) { return wm * WTM + (A_KC ? i * 4 + g : (i & ~1) * 4 + 2 * g + (i & 1)); };
  auto col_of = [&](int j) {
    return wn * WTN + (B_KC ? j * 16 + (lane & 15) : (j & ~1) * 16 + 2 * (lane & 15) + (j & 1));
  };
  if (nsplit > 1) {
    double* __restrict__ W = p.ws + ((int64_t)split * p.ntail + (tile - p.nfull)) * (p.wr * p.wc);
#pragma unroll
    for (int i = 0; i < TMI; ++i)
#pragma unroll
      for (int j = 0; j < TNI; ++j)
        if (row_of(i) < p.wr && col_of(j) < p.wc) W[row_of(i) * p.wc + col_of(j)] = acc[i][j];
    return;
  }
  const int64_t coff = b0 * p.c_b0 + b1 * p.c_b1 + m0 * p.c_m + n0 * p.c_n;
  double* Cg = p.C + coff;
  const double* Ci = p.Cin + coff;
  const int mr = p.M - m0, nr = p.N - n0;
  const double alpha = p.alpha, beta = p.beta;
  if (beta == 0.0) {
#pragma unroll
    for (int i = 0; i < TMI; ++i)
#pragma unroll
      for (int j = 0; j < TNI; ++j)
        if (row_of(i) < mr && col_of(j) < nr) Cg[row_of(i) * p.c_m + col_of(j) * p.c_n] = alpha * acc[i][j];
  } else {
    // the reads of C issued together, before its writes
    double cv[TMI][TNI];
#pragma unroll
    for (int i = 0; i < TMI; ++i)
#pragma unroll
      for (int j = 0; j < TNI; ++j) cv[i][j] = Ci[min(row_of(i), mr - 1) * p.c_m + min(col_of(j), nr - 1) * p.c_n];
#pragma unroll
    for (int i = 0; i < TMI; ++i)
#pragma unroll
      for (int j = 0; j < TNI; ++j)
        if (row_of(i) < mr && col_of(j) < nr)
          Cg[row_of(i) * p.c_m + col_of(j) * p.c_n] = alpha * acc[i][j] + beta * cv[i][j];
  }
}

// C of the tail tiles from their chunk sums, added in chunk order. blockIdx.x:
// tail tile; blockIdx.y and the threads walk its wr x wc elements.
__global__ __launch_bounds__(256) void gemm_f64_reduce(Args p) {
  int b, im, in;
  tile_coords(p, p.nfull + blockIdx.x, &b, &im, &in);
  const int n = p.wr * p.wc;
  const int64_t step = (int64_t)p.ntail * n;
  const double* __restrict__ W = p.ws + (int64_t)blockIdx.x * n;
  const int64_t coff = (b % p.nb0) * p.c_b0 + (b / p.nb0) * p.c_b1;
  for (int e = blockIdx.y * 256 + threadIdx.x; e < n; e += gridDim.y * 256) {
    const int m = im * p.bm + e / p.wc, c = in * p.bn + e % p.wc;
    if (m >= p.M || c >= p.N) continue;
    const int64_t at = coff + m * p.c_m + c * p.c_n;
    const double old = p.beta != 0.0 ? p.Cin[at] : 0.0;
    double acc = 0.0;
    int s = 0;
    for (; s + 4 <= p.ts; s += 4) {  // four chunks' loads in flight
      const double x0 = W[s * step + e], x1 = W[(s + 1) * step + e], x2 = W[(s + 2) * step + e], x3 = W[(s + 3) * step + e];
      acc += x0;
      acc += x1;
      acc += x2;
      acc += x3;
    }
    for (; s < p.ts; ++s) acc += W[s * step + e];
    double v = p.alpha * acc;
    if (p.beta != 0.0) v += p.beta * old;
    p.C[at] = v;
  }
}

// The same for many chunks and few outputs: 16 lanes per output, each adding
// every 16th chunk in increasing order, then the 16 lane sums in order.
__global__ __launch_bounds__(256) void gemm_f64_reduce_wide(Args p) {
  __shared__ double sm[16][17];
  int b, im, in;
  tile_coords(p, p.nfull + blockIdx.x, &b, &im, &in);
  const int n = p.wr * p.wc;
  const int64_t step = (int64_t)p.ntail * n;
  const double* __restrict__ W = p.ws + (int64_t)blockIdx.x * n;
  const int64_t coff = (b % p.nb0) * p.c_b0 + (b / p.nb0) * p.c_b1;
  const int eo = threadIdx.x & 15, sg = threadIdx.x >> 4;
  for (int e0 = blockIdx.y * 16; e0 < n; e0 += gridDim.y * 16) {
    const int e = e0 + eo;
    double acc = 0.0;
    if (e < n) {
      int s = sg;
      for (; s + 48 < p.ts; s += 64) {
        const double x0 = W[s * step + e], x1 = W[(s + 16) * step + e], x2 = W[(s + 32) * step + e],
                     x3 = W[(s + 48) * step + e];
        acc += x0;
        acc += x1;
        acc += x2;
        acc += x3;
      }
      for (; s < p.ts; s += 16) acc += W[s * step + e];
    }
    sm[sg][eo] = acc;
    __syncthreads();
    const int m = im * p.bm + e / p.wc, c = in * p.bn + e % p.wc;
    if (sg == 0 && e < n && m < p.M && c < p.N) {
      double sum = 0.0;
      for (int q = 0; q < 16; ++q) sum += sm[q][eo];
      const int64_t at = coff + m * p.c_m + c * p.c_n;
      double v = p.alpha * sum;
      if (p.beta != 0.0) v += p.beta * p.Cin[at];
      p.C[at] = v;
    }
    __syncthreads();
  }
}

}  // namespace f64pipe
}  // namespace pnk
