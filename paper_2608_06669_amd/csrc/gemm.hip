// Matrix-core GEMM for gfx950 (CDNA4), FP64 / FP32 / BF16 compute.
//
// FP64 products run in gemm_f64_pipe (gemm_f64.hpp), those of a short side and
// a short contraction in gemm_smallk. BF16 and FP32 products of operands stored
// in that type along k run in gemm_pipe, those of at most 32 rows or columns in
// gemm_thin. The others (FP64: an operand contiguous along neither index) run
// in gemm_kernel:
//
// One workgroup = 4 wavefronts of 64 lanes computes a BM x BN tile of C.
// The waves form a WGM x WGN grid; each wave owns (BM/WGM) x (BN/WGN)
// outputs as a grid of matrix-core instruction tiles held in registers for
// the whole K loop. A and B panels of depth BK are staged through two LDS
// buffers: while the matrix cores work on one buffer, the next panel's
// global loads are in flight and are then written to the other buffer, so
// each K step costs one barrier. Global loads are 16-byte vectors along the
// operand's contiguous index whenever strides and alignment allow. Operands
// are converted to the compute type as they are written to LDS, so FP64
// tensors feed the FP32 and BF16 products without a separate cast pass.
//
// Matrix-core instructions and operand layouts (64 lanes, lane l):
//   f64  4x4x4 (4 blocks), used as one 4 x 16 x 4 product:
//        A[i][k] at i = l%4, k = l/16 (the same for the 4 blocks);
//        B[k][j] at j = l%16, k = l/16;  D[i][j] at i = l/16, j = l%16.
//        On gfx950 this instruction runs at the full FP64 matrix rate (75 to
//        77 TFLOP/s with operands in registers), while the 16x16x4 f64
//        instruction reaches 36 to 48.
//   f32  16x16x4:  A[i][k] at i = l%16, k = l/16;  B[k][j] at j = l%16;
//        D[i][j] at j = l%16, i = 4*(l/16) + r, r = 0..3
//   bf16 16x16x32: A[i][k..k+7] at i = l%16, k = 8*(l/16); B likewise;
//        D as f32
//
// Workgroup order: each XCD takes a contiguous range of tiles (hardware
// dispatches block ids round-robin over the 8 XCDs), ordered in groups of 8
// row tiles with the row tile fastest, so the workgroups resident on one
// XCD share their A and B panels in that XCD's L2 (85 % L2 hits on a BF16
// 3600^3 product against 72 % in plain order).
//
// Products with too few output tiles to fill the GPU split the contraction
// (split-K); partial sums are added afterwards in a fixed order, so results
// never depend on timing.

#include "gemm.hpp"
#include "gemm_f64.hpp"
#include "mfma_tiles.hpp"

#include <algorithm>
#include <type_traits>

namespace pnk {
namespace {

using namespace tiles;

struct KArgs {
  int M, N, K, nb0;
  int splits, kchunk;  // split-K: blockIdx.z = zb * splits + split
  double* ws;          // partial sums [split][batch][M][N] when splits > 1
  int nbtot;
  int tiles_m, tiles_n;
  int a_vec, b_vec;    // 16-byte vector loads allowed
  const void* A;
  int64_t a_m, a_k, a_b0, a_b1;
  const void* B;
  int64_t b_k, b_n, b_b0, b_b1;
  const void* A2;  // optional second product A2 B2 (same strides as A, B)
  const void* B2;
  void* C;
  const void* Cin;  // what beta multiplies
  int64_t c_m, c_n, c_b0, c_b1;
  double alpha, beta;
};

template <class Mma, typename TA, typename TB, typename TC, int BM, int BN, int BK, int WGM, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256) void gemm_kernel(KArgs p) {
  using L = typename Mma::L;
  using Acc = typename Mma::Acc;
  constexpr int WGN = 4 / WGM;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TMI = WTM / Mma::TM, TNI = WTN / Mma::TN;
  static_assert(WTM % Mma::TM == 0 && WTN % Mma::TN == 0, "wave tile must split into instruction tiles");
  static_assert(BK % Mma::KSTEP == 0, "BK must be a multiple of the MFMA depth");
  constexpr int PA = kPad, PB = kPad;
  constexpr int ALDS = lds_elems<Mma, BM, BK, PA>();
  constexpr int BLDS = lds_elems<Mma, BN, BK, PB>();
  __shared__ __attribute__((aligned(16))) L As[2][ALDS];
  __shared__ __attribute__((aligned(16))) L Bs[2][BLDS];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WGN;
  const int wn = wave % WGN;

  const int ntiles = p.tiles_m * p.tiles_n;
  int bid = blockIdx.x;
  {
    // XCD x receives block ids x, x + 8, ...: give it the contiguous range
    // of q + (x < r) tiles that starts at x q + min(x, r)
    const int q = ntiles >> 3, r = ntiles & 7, x = bid & 7;
    bid = x * q + min(x, r) + (bid >> 3);
  }
  // tiles in groups of (up to) 8 row tiles: within a group the row tile
  // runs fastest, so the workgroups resident on one XCD share both their A
  // and their B panels in L2 (with the row tile fastest over all rows, each
  // XCD streamed every A panel once per column block)
  constexpr int kGroupM = 8;
  const int gsize = kGroupM * p.tiles_n;
  const int grp = bid / gsize;
  const int first_m = grp * kGroupM;
  const int gm = min(p.tiles_m - first_m, kGroupM);
  const int rem = bid - grp * gsize;
  const int tm = first_m + rem % gm;
  const int tn = rem / gm;
  const int m0 = tm * BM;
  const int n0 = tn * BN;

  const int split = blockIdx.z % p.splits;
  const int zb = blockIdx.z / p.splits;
  const int b0 = blockIdx.y % p.nb0;
  const int b1 = blockIdx.y / p.nb0 + zb * (gridDim.y / p.nb0);
  const int kbeg = split * p.kchunk;
  const int kend = min(p.K, kbeg + p.kchunk);
  const TA* __restrict__ Ag = (const TA*)p.A + b0 * p.a_b0 + b1 * p.a_b1;
  const TB* __restrict__ Bg = (const TB*)p.B + b0 * p.b_b0 + b1 * p.b_b1;
  const bool dual = p.A2 != nullptr;
  const TA* __restrict__ Ag2 = dual ? (const TA*)p.A2 + b0 * p.a_b0 + b1 * p.a_b1 : Ag;
  const TB* __restrict__ Bg2 = dual ? (const TB*)p.B2 + b0 * p.b_b0 + b1 * p.b_b1 : Bg;
  const int64_t coff = b0 * p.c_b0 + b1 * p.c_b1;

  Acc acc[TMI][TNI];
#pragma unroll
  for (int i = 0; i < TMI; ++i)
#pragma unroll
    for (int j = 0; j < TNI; ++j) acc[i][j] = Acc{};

  Panel<Mma, TA, BM, BK, A_KC, PA> pa;
  Panel<Mma, TB, BN, BK, B_KC, PB> pb;
  const bool avec = p.a_vec != 0, bvec = p.b_vec != 0;
  const int64_t a_row = p.a_m, a_kk = p.a_k, b_row = p.b_n, b_kk = p.b_k;

  // panels 0 .. nk1-1 read A, B; with a second product, panels nk1 ..
  // 2 nk1-1 read A2, B2 over the same k range into the same accumulators
  const int nk1 = (kend - kbeg + BK - 1) / BK;
  const int nk = dual ? 2 * nk1 : nk1;
  auto load = [&](int t) {
    const bool second = t >= nk1;
    const int k0 = kbeg + (second ? t - nk1 : t) * BK;
    pa.load(second ? Ag2 : Ag, a_row, a_kk, m0, p.M, k0, kend, avec, tid);
    pb.load(second ? Bg2 : Bg, b_row, b_kk, n0, p.N, k0, kend, bvec, tid);
  };
  if (nk > 0) {
    load(0);
    pa.store(As[0], tid);
    pb.store(Bs[0], tid);
    __syncthreads();
  }
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) load(kt + 1);
    const L* Ac = As[cur];
    const L* Bc = Bs[cur];
#pragma unroll
    for (int ks = 0; ks < BK; ks += Mma::KSTEP) {
      if constexpr (Mma::KCONTIG_LDS) {
        const int kk = ks + 8 * (lane >> 4);
        bf8 af[TMI], bfr[TNI];
#pragma unroll
        for (int i = 0; i < TMI; ++i) {
          const int m = wm * WTM + i * 16 + (lane & 15);
          af[i] = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(&Ac[m * (BK + kPadK) + kk]));
        }
#pragma unroll
        for (int j = 0; j < TNI; ++j) {
          const int n = wn * WTN + j * 16 + (lane & 15);
          bfr[j] = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(&Bc[n * (BK + kPadK) + kk]));
        }
#pragma unroll
        for (int i = 0; i < TMI; ++i)
#pragma unroll
          for (int j = 0; j < TNI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      } else if constexpr (sizeof(L) == 8) {
        const int kk = ks + (lane >> 4);
        double af[TMI], bfr[TNI];
#pragma unroll
        for (int i = 0; i < TMI; ++i) af[i] = Ac[kk * (BM + PA) + wm * WTM + i * 4 + (lane & 3)];
#pragma unroll
        for (int j = 0; j < TNI; ++j) bfr[j] = Bc[kk * (BN + PB) + wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
        for (int i = 0; i < TMI; ++i)
#pragma unroll
          for (int j = 0; j < TNI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[i], bfr[j], acc[i][j], 0, 0, 0);
      } else {
        const int kk = ks + (lane >> 4);
        L af[TMI], bfr[TNI];
#pragma unroll
        for (int i = 0; i < TMI; ++i) af[i] = Ac[kk * (BM + PA) + wm * WTM + i * 16 + (lane & 15)];
#pragma unroll
        for (int j = 0; j < TNI; ++j) bfr[j] = Bc[kk * (BN + PB) + wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
        for (int i = 0; i < TMI; ++i)
#pragma unroll
          for (int j = 0; j < TNI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bfr[j], acc[i][j], 0, 0, 0);
      }
    }
    if (kt + 1 < nk) {
      // the other buffer was last read before the previous barrier
      pa.store(As[cur ^ 1], tid);
      pb.store(Bs[cur ^ 1], tid);
    }
    __syncthreads();
  }

  // epilogue: C = alpha * acc + beta * C, or raw partial sums for split-K
  const double alpha = p.alpha, beta = p.beta;
#pragma unroll
  for (int i = 0; i < TMI; ++i)
#pragma unroll
    for (int j = 0; j < TNI; ++j)
#pragma unroll
      for (int r = 0; r < Mma::NACC; ++r) {
        const int row = (Mma::NACC == 1) ? (lane >> 4) : 4 * (lane >> 4) + r;
        const int gm = m0 + wm * WTM + i * Mma::TM + row;
        const int gn = n0 + wn * WTN + j * Mma::TN + (lane & 15);
        if (gm >= p.M || gn >= p.N) continue;
        if (p.splits > 1) {
          const int64_t b = (int64_t)b1 * p.nb0 + b0;
          p.ws[(((int64_t)split * p.nbtot + b) * p.M + gm) * p.N + gn] = acc_get(acc[i][j], r);
        } else {
          const int64_t at = coff + gm * p.c_m + gn * p.c_n;
          double v = alpha * acc_get(acc[i][j], r);
          if (beta != 0.0) v += beta * load_c<TC>((const TC*)p.Cin + at);
          ((TC*)p.C)[at] = from_acc<TC>(v);
        }
      }
}

// FP32 / BF16 products with at most 32 rows (M; a product with few columns
// comes transposed): one wave per 16 columns and MT 16-row tiles, operands
// straight from memory to registers, rounded there, U steps of 32 (BF16) or 16
// (FP32) k ahead; no LDS, no barrier. The wide operand is read once and used
// by MT instructions. Bound by the loads in flight: those of one BF16 J v at o =
// 20, v = 180 read 2.1 GB in 0.79 ms, from 1.8 to 4.2 TB/s (a copy reaches 4.7),
// the waves waiting for 40 to 70 % of their cycles and the matrix cores busy for
// 1 %. Through LDS in 64 x 64 tiles, mostly padding and one panel in flight, J v
// took 4.79 ms in place of 4.58, at o = 10, v = 90 1059 us in place of 970 (FP32
// 1270 and 1186). 20 x 32400 x 20 in 20 batches takes 171 us with one step
// ahead, 212 with two.
// k order, chunks and roundings are those of gemm_kernel: same results.
template <class Mma, typename TA, typename TB, int MT, int U>
__global__ __launch_bounds__(256, U == 1 ? 4 : 2) void gemm_thin(KArgs p) {
  using L = typename Mma::L;
  constexpr bool bf16 = Mma::KCONTIG_LDS;
  constexpr int E = bf16 ? 8 : 4, KS = 4 * E;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int n0 = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 16;
  if (n0 >= p.N) return;
  const int split = blockIdx.z % p.splits;
  const int zb = blockIdx.z / p.splits;
  const int b0 = blockIdx.y % p.nb0;
  const int b1 = blockIdx.y / p.nb0 + zb * (gridDim.y / p.nb0);
  const int kbeg = split * p.kchunk, kend = min(p.K, kbeg + p.kchunk);
  const int nk1 = (kend - kbeg + KS - 1) / KS, nk = p.A2 ? 2 * nk1 : nk1;
  // (rows and columns past the matrix read its last ones; not written)
  const int col = n0 + (lane & 15);
  const int64_t aoff = b0 * p.a_b0 + b1 * p.a_b1, boff = b0 * p.b_b0 + b1 * p.b_b1 + min(col, p.N - 1) * p.b_n;
  int64_t arow[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) arow[i] = aoff + min(i * 16 + (lane & 15), p.M - 1) * p.a_m;
  struct Raw {
    TA a[MT][E];
    TB b[E];
  };
  auto kofs = [&](int e) { return bf16 ? 8 * g + e : 4 * e + g; };
  auto fetch = [&](auto (&r)[E], auto* x, int64_t s_k, bool vec, int k0) {
    using T = std::remove_reference_t<decltype(r[0])>;
    const T* row = (const T*)x;
    if (k0 + KS <= kend) {
      if (bf16 && vec) {
        const uint4* q = reinterpret_cast<const uint4*>(row + k0 + 8 * g);
#pragma unroll
        for (int u = 0; u < (int)sizeof(r) / 16; ++u) reinterpret_cast<uint4*>(r)[u] = q[u];
        return;
      }
      const T* q = row + (k0 + kofs(0)) * s_k;
      const int64_t st = bf16 ? s_k : 4 * s_k;
#pragma unroll
      for (int e = 0; e < E; ++e) r[e] = q[e * st];
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int k = k0 + kofs(e);
        const T v = row[min(k, kend - 1) * s_k];
        r[e] = k < kend ? v : T(0);
      }
    }
  };
  auto load = [&](Raw& r, int t) {
    t = min(t, nk - 1);
    const bool second = t >= nk1;
    const int k0 = kbeg + (second ? t - nk1 : t) * KS;
    const TA* A = (const TA*)(second ? p.A2 : p.A);
    const TB* B = (const TB*)(second ? p.B2 : p.B);
#pragma unroll
    for (int i = 0; i < MT; ++i) fetch(r.a[i], A + arow[i], p.a_k, p.a_vec != 0, k0);
    fetch(r.b, B + boff, p.b_k, p.b_vec != 0, k0);
  };
  f4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = f4{};
  auto multiply = [&](const Raw& r) {
    if constexpr (bf16) {
      u16x8 x, y;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = to_lds<TB, L>(r.b[e]);
#pragma unroll
      for (int i = 0; i < MT; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = to_lds<TA, L>(r.a[i][e]);
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, x), __builtin_bit_cast(bf8, y), acc[i], 0,
                                                         0, 0);
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_lds<TA, L>(r.a[i][e]), to_lds<TB, L>(r.b[e]), acc[i], 0, 0, 0);
    }
  };
  Raw x[U], y[U];
#pragma unroll
  for (int u = 0; u < U; ++u) load(x[u], u);
  int t = 0;
  for (; t + U < nk; t += 2 * U) {
#pragma unroll
    for (int u = 0; u < U; ++u) load(y[u], t + U + u);
#pragma unroll
    for (int u = 0; u < U; ++u) multiply(x[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) load(x[u], t + 2 * U + u);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + U + u < nk) multiply(y[u]);
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (t + u < nk) multiply(x[u]);

#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = i * 16 + 4 * g + r;
      if (row >= p.M || col >= p.N) continue;
      if (p.splits > 1) {
        const int64_t b = (int64_t)b1 * p.nb0 + b0;
        p.ws[(((int64_t)split * p.nbtot + b) * p.M + row) * p.N + col] = (double)acc[i][r];
      } else {
        const int64_t at = b0 * p.c_b0 + b1 * p.c_b1 + row * p.c_m + col * p.c_n;
        double v = p.alpha * (double)acc[i][r];
        if (p.beta != 0.0) v += p.beta * ((const double*)p.Cin)[at];
        ((double*)p.C)[at] = v;
      }
    }
}

// C[b][m][n] = alpha * sum_s ws[s][b][m][n] + beta * C[b][m][n] (fixed order)
template <typename TC>
__global__ __launch_bounds__(256) void splitk_reduce(KArgs p) {
  const int64_t MN = (int64_t)p.M * p.N;
  const int64_t total = MN * p.nbtot;
  // one row-major output: its address is the element index
  const bool flat = p.nbtot == 1 && p.c_n == 1 && p.c_m == p.N;
  for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    double acc = 0.0;
    // four chunks' loads in flight before they are added, in chunk order
    int s = 0;
    for (; s + 4 <= p.splits; s += 4) {
      const double x0 = p.ws[(int64_t)s * total + e], x1 = p.ws[(int64_t)(s + 1) * total + e];
      const double x2 = p.ws[(int64_t)(s + 2) * total + e], x3 = p.ws[(int64_t)(s + 3) * total + e];
      acc += x0;
      acc += x1;
      acc += x2;
      acc += x3;
    }
    for (; s < p.splits; ++s) acc += p.ws[(int64_t)s * total + e];
    int64_t at = e;
    if (!flat) {
      const int64_t b = e / MN;
      const int m = (int)((e % MN) / p.N), n = (int)(e % p.N);
      const int b0 = (int)(b % p.nb0), b1 = (int)(b / p.nb0);
      at = b0 * p.c_b0 + b1 * p.c_b1 + m * p.c_m + n * p.c_n;
    }
    double v = p.alpha * acc;
    if (p.beta != 0.0) v += p.beta * load_c<TC>((const TC*)p.Cin + at);
    ((TC*)p.C)[at] = from_acc<TC>(v);
  }
}

// The same sum for many splits and few outputs: 16 lanes per output, each
// adding every 16th split in increasing order, then the 16 lane sums in
// order (deterministic, and no lane walks all splits).
template <typename TC>
__global__ __launch_bounds__(256) void splitk_reduce_wide(KArgs p) {
  __shared__ double sm[16][17];
  const int64_t MN = (int64_t)p.M * p.N;
  const int64_t total = MN * p.nbtot;
  const int eo = threadIdx.x & 15, sg = threadIdx.x >> 4;
  for (int64_t e0 = blockIdx.x * (int64_t)16; e0 < total; e0 += (int64_t)gridDim.x * 16) {
    const int64_t e = e0 + eo;
    double acc = 0.0;
    if (e < total)
      for (int s = sg; s < p.splits; s += 16) acc += p.ws[(int64_t)s * total + e];
    sm[sg][eo] = acc;
    __syncthreads();
    if (sg == 0 && e < total) {
      double sum = 0.0;
      for (int g = 0; g < 16; ++g) sum += sm[g][eo];
      const int64_t b = e / MN;
      const int m = (int)((e % MN) / p.N), n = (int)(e % p.N);
      const int b0 = (int)(b % p.nb0), b1 = (int)(b / p.nb0);
      const int64_t at = b0 * p.c_b0 + b1 * p.c_b1 + m * p.c_m + n * p.c_n;
      double v = p.alpha * sum;
      if (p.beta != 0.0) v += p.beta * load_c<TC>((const TC*)p.Cin + at);
      ((TC*)p.C)[at] = from_acc<TC>(v);
    }
    __syncthreads();
  }
}

// Product of two k-contiguous operands in the compute type (rows 16-byte
// aligned; BF16: the contraction a multiple of 64, zero-padded), BM x BN tiles,
// panels of 128 bytes of k (64 BF16, 32 FP32) in a ring of three LDS stages filled straight from global memory
// (16 bytes per lane, no register staging), so two panels' loads are in
// flight while the matrix cores work on the third. A stage holds A then B,
// [row][128 bytes] each; the eight 16-byte chunks of a row are stored at slot
// chunk ^ ((row / 2) % 8), which spreads the fragment reads of 16
// consecutive rows over all 64 banks (each wave's load writes 1 KB
// contiguously: its lanes fetch the chunks in slot order). Each wave forms
// a 64 x 64 block of the tile: BM = 128 with 4 waves (96 KB of LDS), or BM
// = 256 with 8 waves (144 KB: one workgroup per CU, two waves per SIMD; on
// MI355X 1.1-1.4x faster than 128 x 128 on the 3600 x 3600 x 7232, 210 x
// 16290 x 16290 and 400 x 3600 x 32400 products and 1.4x at 8192^3). Same
// tile order, split-K and epilogue as gemm_kernel.
// FP32: 128 x 64 tiles with 4 waves of 64 x 32 (72 KB: two workgroups per CU; 128
// x 128 would leave 2304^2 outputs 1.3 tiles per CU), 16-byte chunks of k past
// the end read as zeros; k in ascending order like gemm_kernel, the same
// results: 2304^3 230 us where the register-staged 128 x 128 tiles took 405.
template <int N>
__device__ inline void wait_vm_lgkm0() {  // vmcnt(N), lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

template <typename T, int BM, int BN, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_pipe(KArgs p) {
  constexpr bool f32 = sizeof(T) == 4;
  constexpr int BK = 128 / (int)sizeof(T), CE = 16 / (int)sizeof(T), STAGES = 3, NT = 64 * NW;
  static_assert(BM == 64 * (NW / 2), "64 rows per wave, two waves across the tile");
  constexpr int WTN = BN / 2, TNJ = WTN / 16;
  constexpr int SE = (BM + BN) * BK;                 // elements per stage
  constexpr int CA = BM * 8 / NT, CB = BN * 8 / NT;  // 16-byte chunks per thread and stage
  __shared__ __attribute__((aligned(1024))) T st0[SE], st1[SE], st2[SE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  const int ntiles = p.tiles_m * p.tiles_n;
  int bid = blockIdx.x;
  {
    const int q = ntiles >> 3, r = ntiles & 7, x = bid & 7;
    bid = x * q + min(x, r) + (bid >> 3);
  }
  constexpr int kGroupM = 8;
  const int gsize = kGroupM * p.tiles_n;
  const int grp = bid / gsize;
  const int first_m = grp * kGroupM;
  const int gm = min(p.tiles_m - first_m, kGroupM);
  const int rem = bid - grp * gsize;
  const int m0 = (first_m + rem % gm) * BM;
  const int n0 = (rem / gm) * BN;

  const int split = blockIdx.z % p.splits;
  const int zb = blockIdx.z / p.splits;
  const int b0 = blockIdx.y % p.nb0;
  const int b1 = blockIdx.y / p.nb0 + zb * (gridDim.y / p.nb0);
  const int kbeg = split * p.kchunk;
  const int klen = min(p.K, kbeg + p.kchunk) - kbeg;
  const int nk = f32 ? (klen + BK - 1) / BK : klen / BK;  // >= 1
  const T* __restrict__ Ag = (const T*)p.A + b0 * p.a_b0 + b1 * p.a_b1 + kbeg;
  const T* __restrict__ Bg = (const T*)p.B + b0 * p.b_b0 + b1 * p.b_b1 + kbeg;
  double* Cg = (double*)p.C + b0 * p.c_b0 + b1 * p.c_b1;
  const double* Ci = (const double*)p.Cin + b0 * p.c_b0 + b1 * p.c_b1;

  // this thread's chunks c = j NT + tid (row c / 8, slot c % 8) of A (j <
  // CA) and of B (j < CB) (rows past the matrix read its last row; those
  // outputs are not written)
  const T* ga[CA];
  const T* gb[CB];
  int ka[CA], kb[CB];  // their k within a panel
#pragma unroll
  for (int j = 0; j < CA; ++j) {
    const int c = j * NT + tid, r = c >> 3, slot = c & 7, g = slot ^ ((r >> 1) & 7);
    ka[j] = CE * g;
    ga[j] = Ag + (int64_t)min(m0 + r, p.M - 1) * p.a_m + CE * g;
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    const int c = j * NT + tid, r = c >> 3, slot = c & 7, g = slot ^ ((r >> 1) & 7);
    kb[j] = CE * g;
    gb[j] = Bg + (int64_t)min(n0 + r, p.N - 1) * p.b_n + CE * g;
  }
  // panel t into stage st (past the last panel: the last one again, never
  // read)
  auto issue = [&](T* st, int t) {
    const int k0 = min(t, nk - 1) * BK;
    auto at = [&](const T* g, int k) -> const void* {
      return !f32 || k0 + k < klen ? (const void*)(g + k0) : (const void*)f64pipe::zero_src;
    };
#pragma unroll
    for (int j = 0; j < CA; ++j)
      f64pipe::to_lds<true>(at(ga[j], ka[j]), (uint32_t*)st + (j * NT + wave * 64) * 4);
#pragma unroll
    for (int j = 0; j < CB; ++j)
      f64pipe::to_lds<true>(at(gb[j], kb[j]), (uint32_t*)(st + BM * BK) + (j * NT + wave * 64) * 4);
  };
  f4 acc[4][TNJ];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < TNJ; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const T* st) {
   if constexpr (f32) {
#pragma unroll
    for (int ks = 0; ks < BK / 4; ++ks) {  // k = 4 ks + lane / 16
      float af[4], bfr[TNJ];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 64 + i * 16 + (lane & 15);
        af[i] = st[row * BK + 4 * (ks ^ ((row >> 1) & 7)) + (lane >> 4)];
      }
#pragma unroll
      for (int j = 0; j < TNJ; ++j) {
        const int row = wn * WTN + j * 16 + (lane & 15);
        bfr[j] = st[BM * BK + row * BK + 4 * (ks ^ ((row >> 1) & 7)) + (lane >> 4)];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < TNJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
   } else {
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      const int q = 4 * ks + (lane >> 4);  // this lane's 8-element chunk of the 32-deep step
      bf8 af[4], bfr[TNJ];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 64 + i * 16 + (lane & 15);
        af[i] = __builtin_bit_cast(bf8, *reinterpret_cast<const u16x8*>(st + row * BK + 8 * (q ^ ((row >> 1) & 7))));
      }
#pragma unroll
      for (int j = 0; j < TNJ; ++j) {
        const int row = wn * WTN + j * 16 + (lane & 15);
        bfr[j] = __builtin_bit_cast(
            bf8, *reinterpret_cast<const u16x8*>(st + BM * BK + row * BK + 8 * (q ^ ((row >> 1) & 7))));
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < TNJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
   }
  };
  issue(st0, 0);
  issue(st1, 1);
  // step t: wait for panel t (CA + CB loads per panel per thread; the next
  // panel's may still be in flight) and for this wave's earlier LDS reads,
  // then a barrier (every wave's share of panel t has landed and every wave
  // is done with the stage about to be refilled), refill that stage with
  // panel t + 2, and compute panel t. (A plain barrier: the workgroup fence
  // of __syncthreads would wait for all loads in flight.)
  auto step = [&](int t, const T* cur, T* nxt) {
    wait_vm_lgkm0<(CA + CB) * (STAGES - 2)>();
    __builtin_amdgcn_s_barrier();
    issue(nxt, t + STAGES - 1);
    compute(cur);
  };
  // panel t sits in stage t % 3. Whole rounds of three in the loop, the
  // rest after it: with steps under a condition inside the loop the compiler
  // no longer tells the stages apart and waits for every load in flight
  // before each LDS read
  int t = 0;
  for (; t + 3 <= nk; t += 3) {
    step(t, st0, st2);
    step(t + 1, st1, st0);
    step(t + 2, st2, st1);
  }
  if (t < nk) step(t, st0, st2);
  if (t + 1 < nk) step(t + 1, st1, st0);
  wait_vm_lgkm0<0>();  // no load still writing LDS when the workgroup ends

  // epilogue (three uniform cases, each straight-line so the compiler can
  // count its memory operations): split-K partial sums; C = alpha acc; C =
  // alpha acc + beta C with the 16 reads of C of a row of tiles issued
  // together before its writes
  const double alpha = p.alpha, beta = p.beta;
  auto row_of = [&](int i, int r) { return m0 + wm * 64 + i * 16 + 4 * (lane >> 4) + r; };
  auto col_of = [&](int j) { return n0 + wn * WTN + j * 16 + (lane & 15); };
  if (p.splits > 1) {
    double* __restrict__ W = p.ws + ((int64_t)split * p.nbtot + (int64_t)b1 * p.nb0 + b0) * p.M * p.N;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < TNJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row_of(i, r) < p.M && col_of(j) < p.N) W[(int64_t)row_of(i, r) * p.N + col_of(j)] = (double)acc[i][j][r];
  } else if (beta == 0.0) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < TNJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row_of(i, r) < p.M && col_of(j) < p.N)
            Cg[row_of(i, r) * p.c_m + col_of(j) * p.c_n] = alpha * (double)acc[i][j][r];
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double cv[TNJ][4];
#pragma unroll
      for (int j = 0; j < TNJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          cv[j][r] = Ci[min(row_of(i, r), p.M - 1) * p.c_m + min(col_of(j), p.N - 1) * p.c_n];
#pragma unroll
      for (int j = 0; j < TNJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row_of(i, r) < p.M && col_of(j) < p.N)
            Cg[row_of(i, r) * p.c_m + col_of(j) * p.c_n] = alpha * (double)acc[i][j][r] + beta * cv[j][r];
    }
  }
}

// Products with a short contraction (K <= kSmallK) and a short output side
// (<= kSmallSide): a matrix-core tile would be mostly padding and the cost
// is one pass over the long operand. Each lane owns one index of the long
// output side, holds its K operand values in registers and produces every
// output along the short side; the short operand is staged in LDS and read
// as broadcasts. LONG_N: the long side is N.
constexpr int kSmallK = 32, kSmallSide = 32;

template <bool LONG_N>
__global__ __launch_bounds__(256) void gemm_smallk(KArgs p) {
  __shared__ double sh[kSmallSide * kSmallK];  // the short operand, [s][k]
  const int b0 = blockIdx.y % p.nb0;
  const int b1 = blockIdx.y / p.nb0 + blockIdx.z * (gridDim.y / p.nb0);
  const double* __restrict__ A = (const double*)p.A + b0 * p.a_b0 + b1 * p.a_b1;
  const double* __restrict__ B = (const double*)p.B + b0 * p.b_b0 + b1 * p.b_b1;
  double* C = (double*)p.C + b0 * p.c_b0 + b1 * p.c_b1;
  const double* Cin = (const double*)p.Cin + b0 * p.c_b0 + b1 * p.c_b1;
  const int L = LONG_N ? p.N : p.M;
  const int S = LONG_N ? p.M : p.N;
  // the short side is split over p.splits groups of workgroups. With at
  // least 8 blocks of 256 along the long side, the groups of one block share
  // an XCD (block ids go round-robin over the 8 XCDs), so its operand is
  // read from HBM once; fewer blocks (batched products) map in order
  const int sgn = p.splits;
  const int nlb = (L + 255) / 256;
  int lblock, sg;
  if (nlb >= 8) {
    const int xcd = (int)(blockIdx.x % 8), q8 = (int)(blockIdx.x / 8);
    lblock = xcd + 8 * (q8 / sgn);
    sg = q8 % sgn;
  } else {
    lblock = (int)blockIdx.x / sgn;
    sg = (int)blockIdx.x % sgn;
  }
  const int sper = (S + sgn - 1) / sgn;
  const int s0 = sg * sper, s1 = min(S, s0 + sper);
  for (int q = threadIdx.x; q < S * p.K; q += 256) {
    const int s = q / p.K, k = q % p.K;
    sh[s * kSmallK + k] = LONG_N ? A[s * p.a_m + k * p.a_k] : B[k * p.b_k + s * p.b_n];
  }
  __syncthreads();
  const int l = lblock * 256 + threadIdx.x;
  if (l >= L || s0 >= s1) return;
  double r[kSmallK];
#pragma unroll
  for (int k = 0; k < kSmallK; ++k)
    r[k] = k < p.K ? (LONG_N ? B[k * p.b_k + l * p.b_n] : A[l * p.a_m + k * p.a_k]) : 0.0;
  for (int s = s0; s < s1; ++s) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kSmallK; ++k)
      if (k < p.K) acc += sh[s * kSmallK + k] * r[k];
    const int64_t at = LONG_N ? s * p.c_m + l * p.c_n : l * p.c_m + s * p.c_n;
    double v = p.alpha * acc;
    if (p.beta != 0.0) v += p.beta * Cin[at];
    C[at] = v;
  }
}

// The batch as gridDim.y gridDim.z, y a multiple of nb0, within the limit of
// both (which a batch has to keep in every kernel, also one that counts its
// workgroups otherwise).
void batch_grid(const GemmDesc& d, int64_t* gy, int64_t* gz) {
  *gy = d.nb0;
  *gz = d.nb1;
  while (*gy * 2 <= 65535 && *gz % 2 == 0) { *gy *= 2; *gz /= 2; }
  PNK_REQUIRE(*gy <= 65535 && *gz <= 65535, "gemm: batch too large");
}

void launch_smallk(const GemmDesc& d, const void* A, const void* B, void* C, hipStream_t s) {
  KArgs p{};
  p.M = d.M; p.N = d.N; p.K = d.K; p.nb0 = d.nb0; p.splits = 1;
  p.A = A; p.a_m = d.a_m; p.a_k = d.a_k; p.a_b0 = d.a_b0; p.a_b1 = d.a_b1;
  p.B = B; p.b_k = d.b_k; p.b_n = d.b_n; p.b_b0 = d.b_b0; p.b_b1 = d.b_b1;
  p.C = C; p.c_m = d.c_m; p.c_n = d.c_n; p.c_b0 = d.c_b0; p.c_b1 = d.c_b1;
  p.Cin = d.Cin ? d.Cin : (double*)C;
  p.alpha = d.alpha; p.beta = d.beta;
  // the long side is the one with more elements; ties go to N (usually the
  // contiguous index of C)
  const bool long_n = d.N >= d.M;
  const int L = long_n ? d.N : d.M;
  const int S = long_n ? d.M : d.N;
  int64_t gy, gz;
  batch_grid(d, &gy, &gz);
  // one lane per index of the long side leaves a few waves per SIMD when
  // the long side is short of a million: split the short side into groups
  // (at most four) until about 4096 waves run
  const int64_t nlb = ceil_div(L, 256);
  const int64_t waves = nlb * 4 * (int64_t)d.nb0 * d.nb1;
  p.splits = (int)std::max<int64_t>(1, std::min<int64_t>({4, S, ceil_div(4096, std::max<int64_t>(waves, 1))}));
  dim3 grid((unsigned)((nlb >= 8 ? 8 * ceil_div(nlb, 8) : nlb) * p.splits), (unsigned)gy, (unsigned)gz);
  if (long_n) gemm_smallk<true><<<grid, 256, 0, s>>>(p);
  else gemm_smallk<false><<<grid, 256, 0, s>>>(p);
  PNK_CHECK_LAUNCH();
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

template <typename T>
bool vec_ok(const void* base, int64_t s_row, int64_t s_k, int64_t s_b0, int64_t s_b1, bool kc) {
  const int64_t V = 16 / (int64_t)sizeof(T);
  if (!aligned16(base) || s_b0 % V != 0 || s_b1 % V != 0) return false;
  if (kc) return s_k == 1 && s_row % V == 0;
  return s_row == 1 && s_k % V == 0;
}

// gemm_thin, transposed if the columns are the few
template <class Mma, typename TA, typename TB>
void launch_thin(const KArgs& p, bool akc, bool bkc, int64_t gy, int64_t gz, hipStream_t s) {
  if (p.M > 32) {
    KArgs q = p;
    std::swap(q.M, q.N);
    q.A = p.B; q.A2 = p.B2; q.a_m = p.b_n; q.a_k = p.b_k; q.a_b0 = p.b_b0; q.a_b1 = p.b_b1; q.a_vec = p.b_vec;
    q.B = p.A; q.B2 = p.A2; q.b_n = p.a_m; q.b_k = p.a_k; q.b_b0 = p.a_b0; q.b_b1 = p.a_b1; q.b_vec = p.a_vec;
    std::swap(q.c_m, q.c_n);
    launch_thin<Mma, TB, TA>(q, bkc, akc, gy, gz, s);
    return;
  }
  KArgs q = p;
  // 16-byte loads along k: rows and batches aligned
  q.a_vec = akc && p.a_vec;
  q.b_vec = bkc && p.b_vec;
  const int waves = (int)std::min<int64_t>(4, ceil_div(p.N, 16));
  const dim3 grid((unsigned)ceil_div(p.N, 16 * waves), (unsigned)gy, (unsigned)(gz * p.splits));
  // a few steps: one ahead, and twice the waves for the registers saved
  const bool brief = (int64_t)p.kchunk * (p.A2 ? 2 : 1) <= 128;
  if (p.M <= 16) {
    if (brief) gemm_thin<Mma, TA, TB, 1, 1><<<grid, 64 * waves, 0, s>>>(q);
    else gemm_thin<Mma, TA, TB, 1, 2><<<grid, 64 * waves, 0, s>>>(q);
  } else if (brief) {
    gemm_thin<Mma, TA, TB, 2, 1><<<grid, 64 * waves, 0, s>>>(q);
  } else {
    gemm_thin<Mma, TA, TB, 2, 2><<<grid, 64 * waves, 0, s>>>(q);
  }
  PNK_CHECK_LAUNCH();
}

template <class Mma, typename TA, typename TB, typename TC, int BM, int BN, int BK, int WGM>
void launch_cfg(const GemmDesc& d, const void* A, const void* B, const void* A2, const void* B2, void* C,
                hipStream_t s) {
  KArgs p;
  p.A2 = A2;
  p.B2 = A2 ? B2 : nullptr;
  p.M = d.M; p.N = d.N; p.K = d.K; p.nb0 = d.nb0;
  p.tiles_m = (int)ceil_div(d.M, BM);
  p.tiles_n = (int)ceil_div(d.N, BN);
  p.A = A; p.a_m = d.a_m; p.a_k = d.a_k; p.a_b0 = d.a_b0; p.a_b1 = d.a_b1;
  p.B = B; p.b_k = d.b_k; p.b_n = d.b_n; p.b_b0 = d.b_b0; p.b_b1 = d.b_b1;
  p.C = C; p.c_m = d.c_m; p.c_n = d.c_n; p.c_b0 = d.c_b0; p.c_b1 = d.c_b1;
  p.Cin = d.Cin ? d.Cin : (double*)C;
  p.alpha = d.alpha; p.beta = d.beta;
  const int64_t nb = (int64_t)d.nb0 * d.nb1;
  p.nbtot = (int)nb;
  const bool akc = d.a_k == 1 && d.a_m != 1;
  const bool bkc = d.b_k == 1 && d.b_n != 1;
  p.a_vec = vec_ok<TA>(A, d.a_m, d.a_k, d.a_b0, d.a_b1, akc) && (!A2 || vec_ok<TA>(A2, d.a_m, d.a_k, d.a_b0, d.a_b1, akc));
  p.b_vec = vec_ok<TB>(B, d.b_n, d.b_k, d.b_b0, d.b_b1, bkc) && (!A2 || vec_ok<TB>(B2, d.b_n, d.b_k, d.b_b0, d.b_b1, bkc));
  constexpr bool f64 = sizeof(typename Mma::L) == 8;
  if (f64) p.a_vec = p.b_vec = 0;  // operands contiguous along neither index
  // split-K when the output tiles cannot fill the GPU
  int splits = 1;
  const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n * nb;
  // (short contractions are not split: the extra pass over the partial sums
  // would cost more than the product). About 900 workgroups in all (3.5 per
  // CU); thin products with a long contraction stay near 512. Long
  // contractions with fewer than 512 tiles (one or two workgroups per CU,
  // each walking thousands of k steps) are split too.
  // (z also carries the chunks)
  int64_t gy, gz;
  batch_grid(d, &gy, &gz);
  const bool thin = d.M <= 64 && d.K >= 1024;
  const int64_t ws_fit =
      d.ws ? std::min<int64_t>(d.ws_elems / std::max<int64_t>(1, nb * d.M * d.N), 65535 / gz) : 0;
  if (d.ws && d.K >= 256 && (tiles < 256 || (tiles < 512 && d.K >= 8192))) {
    int64_t want = ceil_div(thin ? 512 : 900, tiles);
    want = std::min<int64_t>(want, d.K / (2 * BK));
    want = std::min<int64_t>(want, ws_fit);
    want = std::min<int64_t>(want, 256);
    if (want >= 2) splits = (int)want;
  }
  p.kchunk = splits > 1 ? (int)(ceil_div(ceil_div(d.K, splits), BK) * BK) : d.K;
  if (splits > 1) splits = (int)ceil_div(d.K, p.kchunk);  // no empty chunk
  p.splits = splits;
  p.ws = d.ws;
  PNK_REQUIRE(gy <= 65535 && gz * splits <= 65535, "gemm: batch too large");
  dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)gy, (unsigned)(gz * splits));
  // BF16 operands both k-contiguous with whole 64-deep panels (the packed
  // copies): the pipelined kernel
  constexpr bool pipe_cfg = std::is_same<Mma, MmaBF16>::value && std::is_same<TA, uint16_t>::value &&
                            std::is_same<TB, uint16_t>::value && std::is_same<TC, double>::value && BM == 128 &&
                            BN == 128 && BK == 64;
  auto reduce = [&](const KArgs& q) {
    if (q.splits <= 1) return;
    const int64_t total = nb * d.M * d.N;
    if (q.splits >= 32)
      splitk_reduce_wide<TC><<<(unsigned)std::min<int64_t>(ceil_div(total, 16), 8192), 256, 0, s>>>(q);
    else
      splitk_reduce<TC><<<(unsigned)std::min<int64_t>(ceil_div(total, 256), 4096), 256, 0, s>>>(q);
    PNK_CHECK_LAUNCH();
  };
  if constexpr (!f64 && BM == 64) {
    if (std::min(d.M, d.N) <= 32) {
      launch_thin<Mma, TA, TB>(p, akc, bkc, gy, gz, s);
      if (p.splits > 1 && d.M > 32) std::swap(p.c_m, p.c_n), std::swap(p.M, p.N);
      reduce(p);
      return;
    }
  }
  // FP32 operands both k-contiguous, in one piece
  constexpr bool pipe32 = std::is_same<Mma, MmaF32>::value && std::is_same<TA, float>::value &&
                          std::is_same<TB, float>::value && BM == 128;
  if constexpr (pipe32) {
    if (akc && bkc && !A2 && p.a_vec && p.b_vec && splits == 1 && d.K % 4 == 0) {
      KArgs q = p;
      q.tiles_n = (int)ceil_div(d.N, 64);
      gemm_pipe<float, 128, 64, 4><<<dim3((unsigned)(q.tiles_m * q.tiles_n), grid.y, grid.z), 256, 0, s>>>(q);
      PNK_CHECK_LAUNCH();
      return;
    }
  }
  if (pipe_cfg && akc && bkc && !A2 && d.K % 64 == 0 && p.a_vec && p.b_vec && d.M > 128) {
    // more than 128 rows: 256 x 128 tiles with 8 waves, one workgroup per
    // CU. Tiles that cannot fill the GPU take split-K in whole rounds of
    // 256 workgroups where possible (at most 8 chunks of 8 or more panels):
    // the ladder at o = 20, v = 180 (128 tiles) runs in 2 chunks, the T1
    // part (58 tiles) in 4
    KArgs q = p;
    q.tiles_m = (int)ceil_div(d.M, 256);
    const int64_t t2 = (int64_t)q.tiles_m * q.tiles_n * nb;
    int sp = 1;
    if (d.ws && t2 < 256) {
      double best = (double)t2 / 256.0;
      for (int64_t c = 2; c <= 8 && c <= d.K / (64 * 8) && c <= ws_fit; ++c) {
        const int64_t items = t2 * c;
        const double eff = (double)items / (double)(ceil_div(items, 256) * 256);
        if (eff > best + 1e-9) {
          best = eff;
          sp = (int)c;
        }
      }
    }
    q.kchunk = sp > 1 ? (int)(ceil_div(ceil_div(d.K, sp), 64) * 64) : d.K;
    if (sp > 1) sp = (int)ceil_div(d.K, q.kchunk);
    q.splits = sp;
    PNK_REQUIRE(gz * sp <= 65535, "gemm: batch too large");
    dim3 g2((unsigned)(q.tiles_m * q.tiles_n), (unsigned)gy, (unsigned)(gz * sp));
    gemm_pipe<uint16_t, 256, 128, 8><<<g2, 512, 0, s>>>(q);
    PNK_CHECK_LAUNCH();
    reduce(q);
    return;
  }
  if (pipe_cfg && akc && bkc && !A2 && d.K % 64 == 0 && p.a_vec && p.b_vec) {
    gemm_pipe<uint16_t, 128, 128, 4><<<grid, 256, 0, s>>>(p);
  } else if constexpr (f64) gemm_kernel<Mma, TA, TB, TC, BM, BN, BK, WGM, false, false><<<grid, 256, 0, s>>>(p);
  else if (akc && bkc) gemm_kernel<Mma, TA, TB, TC, BM, BN, BK, WGM, true, true><<<grid, 256, 0, s>>>(p);
  else if (akc) gemm_kernel<Mma, TA, TB, TC, BM, BN, BK, WGM, true, false><<<grid, 256, 0, s>>>(p);
  else if (bkc) gemm_kernel<Mma, TA, TB, TC, BM, BN, BK, WGM, false, true><<<grid, 256, 0, s>>>(p);
  else gemm_kernel<Mma, TA, TB, TC, BM, BN, BK, WGM, false, false><<<grid, 256, 0, s>>>(p);
  PNK_CHECK_LAUNCH();
  reduce(p);
}


// ---- FP64: gemm_f64_pipe ----

// An operand's layout for gemm_f64_pipe: contiguous along k (kc) or along its
// row index, the stride of the other index, whether 16-byte loads apply, and
// whether a tile's offsets need 64 bits (rows from 2^22 elements on, or stored
// backwards): 20 x 20 x 4232000 (o = 20, v = 460) takes 3.48 ms, rows of 4176980
// elements with 32-bit offsets 3.29, gemm_kernel's element-wise loads 8.55.
struct F64Layout {
  bool ok, kc, vec, far;
  int64_t ld;
};
F64Layout f64_layout(const void* x, const void* x2, int rows, int K, int64_t s_r, int64_t s_k, int64_t s_b0, int64_t s_b1) {
  F64Layout l;
  l.kc = s_k == 1 || K == 1;
  l.ok = l.kc || s_r == 1 || rows == 1;
  const int64_t ld = l.kc ? s_r : s_k;
  l.ld = (l.kc ? rows : K) == 1 ? 0 : ld;
  l.far = l.ld < 0 || l.ld >= (int64_t(1) << 22);
  l.vec = aligned16(x) && (!x2 || aligned16(x2)) && l.ld % 2 == 0 && s_b0 % 2 == 0 && s_b1 % 2 == 0 &&
          (l.kc ? K : rows) % 2 == 0;
  return l;
}

// How many tiles run in one piece (nfull) and into how many chunks along K
// the others are cut (ts), by the estimated time. In units of one 64 x 64
// tile's whole contraction at full matrix rate on its CU (512 cycles for each
// 8-deep panel, about 0.235 us of a CU's time; 0.27 with 4-byte loads; a 64 x
// 128 tile 0.456), w units of work per CU take w / e with e the share of the
// matrix rate that the c workgroups resident on a CU reach (measured; a
// little less where every one ends at once). Chunk sums cost a launch (5 us)
// and their bytes twice at 4 TB/s. Checked on MI355X against every (nfull, ts)
// that it considers, for 85 products from 64^3 to 3600^3, the ladders of o/v =
// 10/90 to 20/180 and 20 x 20 x 648000 among them: the choice is within 5 % of
// the best for 58 and within 14 % for all but three (128^3 13 us for 10, 91 x
// 5464 x 4192 107 for 90, 1700 x 2200 x 9000 1299 for 1104). 3600^3 takes 1508
// us with its last 177 64 x 64 tiles in four chunks and 1691 in whole tiles; 90
// x 90 x 9000 20 us in 63 chunks and 562 in one piece.
struct F64Plan {
  int64_t nfull;
  int ts;
};
F64Plan f64_plan(int64_t tiles, int bm, int bn, int K, int64_t sum_elems, int64_t ws_elems, bool vec, bool dual) {
  const double unit = (double)ceil_div(K, 8) * (dual ? 2 : 1) * (bn == 128 ? 0.456 : vec ? 0.235 : 0.27) * bm / 64;
  auto rate = [&](int64_t c, bool together) {
    static const double e[2][2][4] = {{{0.50, 0.72, 0.85, 0.90}, {0.50, 0.65, 0.78, 0.82}},
                                      {{0.76, 0.85, 0.90, 0.92}, {0.76, 0.74, 0.85, 0.85}}};
    // (four whole tiles to a CU with a long contraction are slower than that:
    // 190 x 19904 x 16112, 933 tiles, takes 2423 us in one piece and 2126 with
    // the last 165 cut, 250 x 13000 x 9000 1241 and 1055, 960 x 3900 x 16000
    // 2268 and 2015; of seven such products one, 1700 x 2200 x 9000, loses: 1193
    // and 1299)
    if (together && bn == 64 && c >= 4 && K >= 8192) return 0.82;
    return e[bn == 128][together][std::min<int64_t>(c, 4) - 1];
  };
  // tiles to a CU up to which they are taken to end together. Four 64 x 64 or
  // three 72 x 64 tiles fit one. Of 64 x 128 tiles and, by registers, 80 x 64
  // ones three and two fit, but with those counts here, in the rates and below
  // the choice was no better for any of 80 products and worse for 2304^3 (433 us
  // in place of 382): the rates above were fitted with these.
  const int64_t resident = bm > 64 ? 3 : 4;
  F64Plan best{tiles, 1};
  const int64_t c0 = ceil_div(tiles, 256);
  double t_best = c0 <= resident ? c0 / rate(c0, true) * unit : ((tiles / 256) / 0.9 + (tiles % 256 ? 1.0 / 0.6 : 0.0)) * unit;
  if (K < 64 || ws_elems <= 0) return best;
  static const int kCuts[] = {2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024};
  const int64_t whole = tiles / 256 * 256;
  const int64_t fulls[3] = {0, whole, whole - 256};
  for (int q = 0; q < 3; ++q) {
    const int64_t nfull = fulls[q], tail = tiles - nfull;
    if (nfull < 0 || tail == 0 || (q > 0 && nfull == 0)) continue;
    for (int ts : kCuts) {
      if ((int64_t)ts * 32 > K || ts * tail * sum_elems > ws_elems) break;
      const int64_t items = tail * ts;
      const double w = (double)(nfull / 256) +
                       (nfull + items > 1024 ? items / 256.0 + 0.3 : (double)ceil_div(items, 256)) / ts +
                       (nfull == 256 ? 0.35 : nfull == 512 ? 0.1 : 0.0);  // (whole tiles outlast the chunks)
      const double t = w / rate(ceil_div(nfull + items, 256), false) * unit + 5.0 + (double)items * sum_elems * 16.0 / 4e6;
      if (t < 0.98 * t_best) {
        t_best = t;
        best = F64Plan{nfull, ts};
      }
    }
  }
  return best;
}

template <int BN, bool A_KC, bool B_KC, bool LONG = false, bool ASC = !A_KC && !B_KC>
void launch_f64_layout(const f64pipe::Args& p, bool vec, dim3 grid, hipStream_t s) {
  if (vec) f64pipe::gemm_f64_pipe<64, BN, A_KC, B_KC, true, LONG, ASC><<<grid, 256, 0, s>>>(p);
  else f64pipe::gemm_f64_pipe<64, BN, A_KC, B_KC, false, LONG, ASC><<<grid, 256, 0, s>>>(p);
}

// LONG: the tile kept to 64 x 64
template <int BN, bool LONG>
void launch_f64_kernel(const f64pipe::Args& p, bool akc, bool bkc, bool vec, bool asc, dim3 grid, hipStream_t s) {
  if (akc && bkc) launch_f64_layout<BN, true, true, LONG>(p, vec, grid, s);
  else if (akc && BN == 64 && asc) launch_f64_layout<64, true, false, LONG, true>(p, vec, grid, s);
  else if (akc) launch_f64_layout<BN, true, false, LONG>(p, vec, grid, s);
  else if (bkc) launch_f64_layout<BN, false, true, LONG>(p, vec, grid, s);
  else launch_f64_layout<BN, false, false, LONG>(p, vec, grid, s);
}

// Rows of a tile for M rows: the count that pads least, 64 if another saves less
// than 5 %. Only for A contiguous along k and B along n in 16-byte loads (the
// products of a few pair rows or occupied rows with a wide operand), and 64
// columns: of 72 x 128 tiles only two fit a CU. (96 x 64 tiles, three to a CU,
// took 72 us where two of 48 rows take 64, 91 x 5464 x 4192.)
int f64_rows(int M, const F64Layout& la, const F64Layout& lb) {
  int best = 64;
  if (!la.kc || lb.kc || !la.vec || !lb.vec || la.far || lb.far) return best;
  static const int kRows[] = {72, 80, 48};
  int64_t pad = ceil_div(M, 64) * 64 * 95 / 100;
  for (int r : kRows) {
    const int64_t q = ceil_div(M, r) * r;
    if (q < pad) {
      pad = q;
      best = r;
    }
  }
  return best;
}

template <int BN>
void launch_f64_tiles(f64pipe::Args p, const F64Layout& la, const F64Layout& lb, int64_t nb, int64_t ws_elems, bool asc,
                      hipStream_t s) {
  const bool vec = la.vec && lb.vec;
  p.bm = BN == 128 || asc ? 64 : f64_rows(p.M, la, lb);
  p.bn = BN;
  p.tm = (int)ceil_div(p.M, p.bm);
  p.tn = (int)ceil_div(p.N, BN);
  p.wr = std::min(p.M, p.bm);
  p.wc = std::min(p.N, BN);
  const int64_t tiles = (int64_t)p.tm * p.tn * nb;
  const F64Plan plan = asc ? F64Plan{tiles, 1} : f64_plan(tiles, p.bm, BN, p.K, (int64_t)p.wr * p.wc, ws_elems, vec, p.A2 != nullptr);
  PNK_REQUIRE(tiles * plan.ts < (int64_t(1) << 31), "gemm: batch too large");
  p.kchunk = plan.ts > 1 ? (int)(ceil_div(ceil_div(p.K, plan.ts), 8) * 8) : p.K;
  p.ts = (int)ceil_div(p.K, p.kchunk);  // no empty chunk
  p.nfull = (int)(p.ts > 1 ? plan.nfull : tiles);
  p.ntail = (int)(tiles - p.nfull);
  const int64_t items = p.nfull + (int64_t)p.ntail * p.ts;
  const dim3 grid((unsigned)std::min(items, f64pipe::kMaxGridX), (unsigned)ceil_div(items, f64pipe::kMaxGridX));
  if (p.bm == 72) f64pipe::gemm_f64_pipe<72, 64, true, false, true><<<grid, 256, 0, s>>>(p);
  else if (p.bm == 80) f64pipe::gemm_f64_pipe<80, 64, true, false, true><<<grid, 256, 0, s>>>(p);
  else if (p.bm == 48) f64pipe::gemm_f64_pipe<48, 64, true, false, true><<<grid, 256, 0, s>>>(p);
  else if (BN == 64 && (la.far || lb.far)) launch_f64_kernel<64, true>(p, la.kc, lb.kc, vec, asc, grid, s);
  else launch_f64_kernel<BN, false>(p, la.kc, lb.kc, vec, asc, grid, s);
  PNK_CHECK_LAUNCH();
  if (p.ntail) {
    const int n = p.wr * p.wc;
    if (p.ts >= 32)
      f64pipe::gemm_f64_reduce_wide<<<dim3((unsigned)p.ntail, (unsigned)ceil_div(n, 16)), 256, 0, s>>>(p);
    else
      f64pipe::gemm_f64_reduce<<<dim3((unsigned)p.ntail, (unsigned)ceil_div(n, 256)), 256, 0, s>>>(p);
    PNK_CHECK_LAUNCH();
  }
}

// False if an operand is contiguous along neither index.
bool launch_f64(const GemmDesc& d, const double* A, const double* B, const double* A2, const double* B2, double* C,
                hipStream_t s) {
  const F64Layout la = f64_layout(A, A2, d.M, d.K, d.a_m, d.a_k, d.a_b0, d.a_b1);
  const F64Layout lb = f64_layout(B, B2, d.N, d.K, d.b_n, d.b_k, d.b_b0, d.b_b1);
  if (!la.ok || !lb.ok) return false;
  int64_t gy, gz;
  batch_grid(d, &gy, &gz);
  f64pipe::Args p{};
  p.M = d.M; p.N = d.N; p.K = d.K; p.nb0 = d.nb0;
  p.A = A; p.B = B; p.A2 = A2; p.B2 = A2 ? B2 : nullptr;
  p.lda = la.ld; p.a_b0 = d.a_b0; p.a_b1 = d.a_b1;
  p.ldb = lb.ld; p.b_b0 = d.b_b0; p.b_b1 = d.b_b1;
  p.C = C; p.c_m = d.c_m; p.c_n = d.c_n; p.c_b0 = d.c_b0; p.c_b1 = d.c_b1;
  p.Cin = d.Cin ? d.Cin : (double*)C;
  p.alpha = d.alpha; p.beta = d.beta;
  p.ws = d.ws;
  const int64_t nb = (int64_t)d.nb0 * d.nb1, ws = d.ws ? d.ws_elems : 0;
  const bool asc = d.ascending && !lb.kc;
  // 64 x 128 tiles read LDS and L2 less for each flop: where the largest
  // products run at the rate that the instruction alone sustains (72 TFLOP/s),
  // 1 to 6 % faster (3600^3 1430 against 1505 us, 2304^3 393 against 420, 1280 x
  // 4096 x 4096 676 against 718). Their coarser rounds cost more than that below
  // about 1e10 multiplications (600 x 3600 x 3600 321 against 310, 2000 x 2000
  // x 2100 321 against 291), and mostly below 512 of them, two to a CU (190 x
  // 19904 x 16112, 468, 2290 against 2140; 1800 x 1800 x 8192, 435, 1084 against
  // 940; but 400 x 3600 x 32400, 203, 1675 against 1890). At 512 to 620 they gain
  // in some products and lose in others, 8 % at most.
  const int64_t tiles128 = ceil_div(d.M, 64) * ceil_div(d.N, 128) * nb;
  const bool wide = !asc && !la.far && !lb.far && f64_rows(d.M, la, lb) == 64 && d.K >= 2048 && tiles128 >= 512 &&
                    (double)d.M * d.N * d.K * nb >= 1e10;
  if (wide) launch_f64_tiles<128>(p, la, lb, nb, ws, asc, s);
  else launch_f64_tiles<64>(p, la, lb, nb, ws, asc, s);
  return true;
}

// Tile choice. FP32/BF16: 128 x 128. Small products: 64 x 64 (split-K fills
// the GPU). FP64: gemm_f64_pipe; an operand contiguous along neither index
// takes the register-staged 64 x 64 kernel.
template <class Mma, typename TA, typename TB, typename TC, int BK>
void launch_sized(const GemmDesc& d, const void* A, const void* B, const void* A2, const void* B2, void* C,
                  hipStream_t s) {
  const int64_t nb = (int64_t)d.nb0 * d.nb1;
  if constexpr (sizeof(typename Mma::L) == 8) {
    if (!launch_f64(d, (const double*)A, (const double*)B, (const double*)A2, (const double*)B2, (double*)C, s))
      launch_cfg<Mma, TA, TB, TC, 64, 64, BK, 2>(d, A, B, A2, B2, C, s);
  } else {
    const int64_t big = ceil_div(d.M, 128) * ceil_div(d.N, 128) * nb;
    // BF16 128 x 128 tiles take two matrix-core steps per panel (64-deep):
    // 25-45 % faster than one on the ring, ladder and T1-ladder products
    constexpr bool bf16 = std::is_same<Mma, MmaBF16>::value;
    constexpr int BK128 = bf16 ? 64 : BK;
    // (BF16 with a long contraction takes them from 64 tiles on, split-K
    // filling the GPU: 1.2-2.3x faster than 64 x 64 on the T1 part of the
    // ladder and the antisymmetric ladder at o = 20, v = 180)
    // (BF16 products the pipelined kernel takes, two packed operands with
    // whole panels: from 32 tiles on, split-K filling the GPU)
    const bool pipe_ok = bf16 && std::is_same<TA, uint16_t>::value && std::is_same<TB, uint16_t>::value &&
                         d.a_k == 1 && d.b_k == 1 && d.K % 64 == 0 && !A2;
    const bool wide = big >= 256 || (bf16 && d.K >= 8192 && big >= 64) || (pipe_ok && big >= 32);
    if (d.M >= 64 && d.N >= 96 && wide) launch_cfg<Mma, TA, TB, TC, 128, 128, BK128, 2>(d, A, B, A2, B2, C, s);
    else launch_cfg<Mma, TA, TB, TC, 64, 64, BK, 2>(d, A, B, A2, B2, C, s);
  }
}

}  // namespace

namespace {

// Rounds one FP64 operand of a (batched) product to the compute type and
// writes it as rows contiguous along k: out[b][r][koff + k] (row length
// ld) = in[b0 * s_b0 + b1 * s_b1 + r * s_r + k * s_k], b = b1 * nb0 + b0.
// 32 x 32 tiles through LDS, so reads are coalesced along whichever index
// is contiguous in the input and writes along k.
struct PackArgs {
  const double* in;
  int64_t s_r, s_k, s_b0, s_b1;
  int rows, K, kz, nb0, ld, koff;  // columns koff .. koff + kz - 1 written, zeros past K
  void* out;
  int vst;  // rows of out 16-byte aligned at every multiple of 8 columns (16-byte stores)
};

template <typename T>
__global__ __launch_bounds__(256) void pack_operand(PackArgs p) {
  // 32 rows x 64 k per workgroup: read coalesced along whichever index is
  // contiguous in the input, then 8 lanes per row write 8 consecutive k
  // each (one 16-byte store of BF16, two of FP32, where aligned)
  __shared__ double tile[64][33];  // [k - k0][r - r0]
  const int tiles_k = (p.kz + 63) / 64;
  const int r0 = (blockIdx.x / tiles_k) * 32, k0 = (blockIdx.x % tiles_k) * 64;
  const int b = blockIdx.y;
  const int b0 = b % p.nb0, b1 = b / p.nb0;
  const double* in = p.in + b0 * p.s_b0 + b1 * p.s_b1;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  if (p.s_r == 1 && p.s_k != 1) {
    // consecutive lanes walk r
    for (int j = ty; j < 64; j += 8) {
      const int r = r0 + tx, k = k0 + j;
      tile[j][tx] = r < p.rows && k < p.K ? in[(int64_t)r + (int64_t)k * p.s_k] : 0.0;
    }
  } else {
    // consecutive lanes walk k
    for (int j = ty; j < 32; j += 8)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int r = r0 + j, k = k0 + 32 * h + tx;
        tile[32 * h + tx][j] = r < p.rows && k < p.K ? in[(int64_t)r * p.s_r + (int64_t)k * p.s_k] : 0.0;
      }
  }
  __syncthreads();
  const int rr = threadIdx.x >> 3, kc = (threadIdx.x & 7) * 8;
  const int r = r0 + rr;
  if (r >= p.rows) return;
  T y[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = to_lds<double, T>(tile[kc + e][rr]);
  T* dst = (T*)p.out + (int64_t)b * p.rows * p.ld + (int64_t)r * p.ld + p.koff + k0 + kc;
  if (p.vst && k0 + kc + 8 <= p.kz) {
    uint4* d4 = reinterpret_cast<uint4*>(dst);
#pragma unroll
    for (int q = 0; q < (int)sizeof(y) / 16; ++q) {
      uint4 w;
      __builtin_memcpy(&w, reinterpret_cast<const char*>(y) + 16 * q, 16);
      d4[q] = w;
    }
  } else {
    for (int e = 0; e < 8 && k0 + kc + e < p.kz; ++e) dst[e] = y[e];
  }
}

// The same rounding for an input already contiguous along k (s_k = 1),
// with 16-byte aligned rows and segments: no transpose, so each lane reads
// 16 / sizeof(T) consecutive doubles of a row and writes them as one
// 16-byte store. Lanes walk the row's chunks, rows follow each other in the
// grid-stride. (Measured on MI355X against a form with one 16-byte load and
// one pair store per lane, fully coalesced: about 5 % faster on the 3600 x
// 3600 operands of the ring products.)
template <typename T>
__global__ __launch_bounds__(256) void pack_operand_kc(PackArgs p) {
  constexpr int VE = 16 / (int)sizeof(T);  // elements per 16-byte store
  const int b = blockIdx.y;
  const int b0 = b % p.nb0, b1 = b / p.nb0;
  const double* __restrict__ in = p.in + b0 * p.s_b0 + b1 * p.s_b1;
  T* __restrict__ out = (T*)p.out + (int64_t)b * p.rows * p.ld + p.koff;
  const int cpr = (p.kz + VE - 1) / VE;  // chunks per row
  const int64_t total = (int64_t)p.rows * cpr;
  for (int64_t c = blockIdx.x * (int64_t)256 + threadIdx.x; c < total; c += (int64_t)gridDim.x * 256) {
    const int r = (int)(c / cpr), k0 = (int)(c % cpr) * VE;
    const double* src = in + (int64_t)r * p.s_r + k0;
    double x[VE];
    if (k0 + VE <= p.K) {
#pragma unroll
      for (int e = 0; e < VE; e += 2) {
        const double2 t = *reinterpret_cast<const double2*>(src + e);
        x[e] = t.x;
        x[e + 1] = t.y;
      }
    } else {
#pragma unroll
      for (int e = 0; e < VE; ++e) x[e] = k0 + e < p.K ? src[e] : 0.0;
    }
    T y[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) y[e] = to_lds<double, T>(x[e]);
    T* dst = out + (int64_t)r * p.ld + k0;
    if (k0 + VE <= p.kz) {
      uint4 w;
      __builtin_memcpy(&w, y, 16);
      *reinterpret_cast<uint4*>(dst) = w;
    } else {
      for (int e = 0; k0 + e < p.kz; ++e) dst[e] = y[e];
    }
  }
}

template <typename T>
void pack(const double* in, int64_t s_r, int64_t s_k, int64_t s_b0, int64_t s_b1, int rows, int K, int kz, int nb0,
          int nb1, int ld, int koff, void* out, hipStream_t s) {
  const int vst = ((uintptr_t)out & 15u) == 0 && ld % 8 == 0 && koff % 8 == 0;
  PackArgs p{in, s_r, s_k, s_b0, s_b1, rows, K, kz, nb0, ld, koff, out, vst};
  // k-contiguous input with 16-byte aligned chunks in and out
  constexpr int VE = 16 / (int)sizeof(T);
  const bool kc = s_k == 1 && rows > 0 && ((uintptr_t)in & 15u) == 0 && s_r % 2 == 0 && s_b0 % 2 == 0 &&
                  s_b1 % 2 == 0 && ((uintptr_t)out & 15u) == 0 && ld % VE == 0 && koff % VE == 0;
  if (kc) {
    const int64_t total = (int64_t)rows * ceil_div(kz, VE);
    dim3 grid((unsigned)std::min<int64_t>(ceil_div(total, 256), 4096), (unsigned)(nb0 * nb1));
    pack_operand_kc<T><<<grid, 256, 0, s>>>(p);
  } else {
    dim3 grid((unsigned)(ceil_div(rows, 32) * ceil_div(kz, 64)), (unsigned)(nb0 * nb1));
    pack_operand<T><<<grid, 256, 0, s>>>(p);
  }
  PNK_CHECK_LAUNCH();
}

void gemm_impl(const GemmDesc& d, const void* A, const void* B, const void* A2, const void* B2, Prec ap, Prec bp,
               void* C, Prec cp, Prec compute, hipStream_t s);

// FP32/BF16 product with FP64 operands rounded once into d.cast_ws (both
// products of a dual call side by side along k). Returns false when it does
// not apply or does not fit.
bool gemm_precast(const GemmDesc& d, const void* A, const void* B, const void* A2, const void* B2, Prec ap, Prec bp,
                  void* C, Prec cp, Prec compute, hipStream_t s) {
  if (!d.cast_ws || (compute != Prec::F32 && compute != Prec::BF16)) return false;
  // an operand is rounded once only when more than one column (row) of
  // tiles reads it; a thin product (the o x o outputs of the Fock terms)
  // streams it once, and rounding it on load saves a pass over it
  const bool pa = ap == Prec::F64 && d.N > 64, pb = bp == Prec::F64 && d.M > 64;
  if (!pa && !pb) return false;
  const int64_t nb = (int64_t)d.nb0 * d.nb1;
  if ((double)d.M * d.N * d.K * nb < 1e7) return false;  // small: convert on load
  const bool dual = A2 != nullptr;
  if (dual && pa != pb) return false;
  const int64_t es = compute == Prec::BF16 ? 2 : 4;
  const int kt = dual ? 2 * d.K : d.K;
  // rows of the copies start on 16-byte boundaries (vector loads); BF16
  // rows are zero-padded to a multiple of 64 elements (whole panels of the
  // pipelined kernel)
  const int lq = compute == Prec::BF16 ? 64 : 16 / (int)es;
  const int ld = (int)((kt + lq - 1) / lq * lq);
  const int64_t need = es * nb * ((pa ? (int64_t)d.M * ld : 0) + (pb ? (int64_t)d.N * ld : 0)) + 256;
  if (need > d.cast_ws_bytes) return false;
  char* base = (char*)d.cast_ws;
  char* abuf = base;
  char* bbuf = base + (((pa ? es * nb * (int64_t)d.M * ld : 0) + 255) & ~int64_t(255));
  GemmDesc e = d;
  e.cast_ws = nullptr;
  const void *An = A, *Bn = B;
  Prec apn = ap, bpn = bp;
  // (the last segment of a row also writes the zeros up to ld)
  auto run_pack = [&](const void* src, bool is_a, int koff, void* dst) {
    const double* in = (const double*)src;
    const int rows = is_a ? d.M : d.N;
    const int64_t sr = is_a ? d.a_m : d.b_n, sk = is_a ? d.a_k : d.b_k;
    const int64_t sb0 = is_a ? d.a_b0 : d.b_b0, sb1 = is_a ? d.a_b1 : d.b_b1;
    const int kz = koff + d.K == kt ? ld - koff : d.K;
    if (es == 2) pack<uint16_t>(in, sr, sk, sb0, sb1, rows, d.K, kz, d.nb0, d.nb1, ld, koff, dst, s);
    else pack<float>(in, sr, sk, sb0, sb1, rows, d.K, kz, d.nb0, d.nb1, ld, koff, dst, s);
  };
  if (pa) {
    run_pack(A, true, 0, abuf);
    if (dual) run_pack(A2, true, d.K, abuf);
    An = abuf;
    apn = compute;
    e.a_m = ld; e.a_k = 1; e.a_b0 = (int64_t)d.M * ld; e.a_b1 = (int64_t)d.nb0 * d.M * ld;
  }
  if (pb) {
    run_pack(B, false, 0, bbuf);
    if (dual) run_pack(B2, false, d.K, bbuf);
    Bn = bbuf;
    bpn = compute;
    e.b_n = ld; e.b_k = 1; e.b_b0 = (int64_t)d.N * ld; e.b_b1 = (int64_t)d.nb0 * d.N * ld;
  }
  // both products of a dual call packed along k: one product of depth 2K;
  // with both operands zero-padded to ld the contraction runs over the
  // padding too
  const bool bpad = !pb && bp == compute && d.b_k == 1 && d.b_kzero >= ld;
  e.K = pa && (pb || bpad) ? ld : kt;
  gemm_impl(e, An, Bn, nullptr, nullptr, apn, bpn, C, cp, compute, s);
  return true;
}

void gemm_impl(const GemmDesc& d, const void* A, const void* B, const void* A2, const void* B2, Prec ap, Prec bp,
               void* C, Prec cp, Prec compute, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.nb0 <= 0 || d.nb1 <= 0) return;
  PNK_REQUIRE(cp == Prec::F64 || cp == Prec::F32, "gemm: C must be f64 or f32");
  PNK_REQUIRE(d.K > 0, "gemm: K must be positive");
  if (gemm_precast(d, A, B, A2, B2, ap, bp, C, cp, compute, s)) return;
#define PNK_GEMM_CASE(MMA, TA, TB, TC, BK) return launch_sized<MMA, TA, TB, TC, BK>(d, A, B, A2, B2, C, s)
  if (compute == Prec::F64) {
    PNK_REQUIRE(ap == Prec::F64 && bp == Prec::F64, "gemm: f64 compute needs f64 operands");
    PNK_REQUIRE(cp == Prec::F64, "gemm: f64 compute writes f64");
    if (d.K <= kSmallK && std::min(d.M, d.N) <= kSmallSide) {
      launch_smallk(d, A, B, C, s);
      if (A2) {
        GemmDesc e = d;
        e.beta = 1.0;
        e.Cin = nullptr;
        launch_smallk(e, A2, B2, C, s);
      }
      return;
    }
    PNK_GEMM_CASE(MmaF64, double, double, double, 16);
  }
  if (compute == Prec::F32) {
    PNK_REQUIRE(cp == Prec::F64, "gemm: f32 compute writes f64");
    if (ap == Prec::F64 && bp == Prec::F64) PNK_GEMM_CASE(MmaF32, double, double, double, 16);
    if (ap == Prec::F64 && bp == Prec::F32) PNK_GEMM_CASE(MmaF32, double, float, double, 16);
    if (ap == Prec::F32 && bp == Prec::F64) PNK_GEMM_CASE(MmaF32, float, double, double, 16);
    if (ap == Prec::F32 && bp == Prec::F32) PNK_GEMM_CASE(MmaF32, float, float, double, 16);
  }
  if (compute == Prec::BF16) {
    PNK_REQUIRE(cp == Prec::F64, "gemm: bf16 compute writes f64");
    if (ap == Prec::F64 && bp == Prec::F64) PNK_GEMM_CASE(MmaBF16, double, double, double, 32);
    if (ap == Prec::F64 && bp == Prec::BF16) PNK_GEMM_CASE(MmaBF16, double, uint16_t, double, 32);
    if (ap == Prec::BF16 && bp == Prec::F64) PNK_GEMM_CASE(MmaBF16, uint16_t, double, double, 32);
    if (ap == Prec::BF16 && bp == Prec::BF16) PNK_GEMM_CASE(MmaBF16, uint16_t, uint16_t, double, 32);
  }
#undef PNK_GEMM_CASE
  PNK_REQUIRE(false, "gemm: unsupported precision combination");
}

}  // namespace

void gemm(const GemmDesc& d, const void* A, Prec ap, const void* B, Prec bp, void* C, Prec cp, Prec compute,
          hipStream_t s) {
  gemm_impl(d, A, B, nullptr, nullptr, ap, bp, C, cp, compute, s);
}

void gemm_sum(const GemmDesc& d, const void* A1, const void* B1, const void* A2, const void* B2, Prec ap, Prec bp,
              void* C, Prec cp, Prec compute, hipStream_t s) {
  PNK_REQUIRE(A2 && B2, "gemm_sum: second product missing");
  gemm_impl(d, A1, B1, A2, B2, ap, bp, C, cp, compute, s);
}

}  // namespace pnk
