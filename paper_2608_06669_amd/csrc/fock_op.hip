// Fock operator A_F in two launches (see fock_op.hpp).
//
// Virtual kernel: one workgroup computes a bm x bm block (a, b) of
// y_ij = f_vv x_ij + x_ij f_vv for one occupied pair (i, j). The two
// contractions form a single matrix-core product over a contraction of
// length 2v: panels 0 .. nkp-1 multiply f_vv[a][c] by x_ij[c][b], panels
// nkp .. 2nkp-1 multiply x_ij[a][c] by f_vv[c][b] (f_vv is symmetric), so
// both accumulate into the same registers (FP64 4x4x4 matrix-core
// instruction, LDS double buffering).
//
// Occupied kernel: the two occupied contractions are short (length o) but
// touch o slices of x per output; done per output they re-read x 2o times.
// Instead one workgroup stages x[:, :, chunk] (all o^2 pairs for a chunk of
// ch consecutive (a, b)) in LDS once and forms both sums for every pair
// from there, so x is read from memory once. The same launch adds the
// virtual part. Trailing workgroups compute the singles, 16 lanes per output.

#include "fock_op.hpp"
#include "mfma_tiles.hpp"

#include <algorithm>

namespace pnk {
namespace {

using namespace tiles;

struct VirArgs {
  int v, tiles_m, tiles, units, per_xcd;
  int vec;  // 16-byte operand loads allowed
  const double* f_vv;
  const double* x2;
  double* y2;
};

template <int BM, int WGM, int BK>
__global__ __launch_bounds__(256) void fock_vir_kernel(VirArgs p) {
  using Mma = MmaF64;
  constexpr int BN = BM;
  constexpr int WGN = 4 / WGM;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TMI = WTM / Mma::TM, TNI = WTN / Mma::TN;
  static_assert(WTM % Mma::TM == 0 && WTN % Mma::TN == 0, "wave tile must split into instruction tiles");
  constexpr int ALDS = lds_elems<Mma, BM, BK>();
  constexpr int BLDS = lds_elems<Mma, BN, BK>();
  __shared__ __attribute__((aligned(16))) double As[2][ALDS];
  __shared__ __attribute__((aligned(16))) double Bs[2][BLDS];

  const int v = p.v;
  const int64_t vv = (int64_t)v * v;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  // Workgroups are dispatched round-robin over the 8 XCDs; consecutive
  // units (the tiles of one pair) are given to one XCD so the pair's slab
  // of x is fetched into that XCD's L2 once.
  const int u = (int)(blockIdx.x % 8) * p.per_xcd + (int)(blockIdx.x / 8);
  if (u >= p.units) return;
  const int pair = u / p.tiles, tile = u % p.tiles;
  const int m0 = (tile % p.tiles_m) * BM;
  const int n0 = (tile / p.tiles_m) * BN;
  const double* __restrict__ X = p.x2 + (int64_t)pair * vv;
  const double* __restrict__ F = p.f_vv;
  const bool vec = p.vec != 0;
  const int nkp = (v + BK - 1) / BK;
  const int nk = 2 * nkp;

  double acc[TMI][TNI];
#pragma unroll
  for (int a = 0; a < TMI; ++a)
#pragma unroll
    for (int b = 0; b < TNI; ++b) acc[a][b] = 0.0;

  Panel<Mma, double, BM, BK, true> pa;   // A[a][c], contiguous along c
  Panel<Mma, double, BN, BK, false> pb;  // B[c][b], contiguous along b
  auto load = [&](int t) {
    const int ph = t >= nkp ? 1 : 0;
    const int k0 = (t - ph * nkp) * BK;
    pa.load(ph ? X : F, v, 1, m0, v, k0, v, vec, tid);
    pb.load(ph ? F : X, 1, v, n0, v, k0, v, vec, tid);
  };
  load(0);
  pa.store(As[0], tid);
  pb.store(Bs[0], tid);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) load(kt + 1);
    const double* Ac = As[cur];
    const double* Bc = Bs[cur];
#pragma unroll
    for (int ks = 0; ks < BK; ks += Mma::KSTEP) {
      const int kk = ks + (lane >> 4);
      double af[TMI], bf[TNI];
#pragma unroll
      for (int a = 0; a < TMI; ++a) af[a] = Ac[kk * (BM + kPad) + wm * WTM + a * 4 + (lane & 3)];
#pragma unroll
      for (int b = 0; b < TNI; ++b) bf[b] = Bc[kk * (BN + kPad) + wn * WTN + b * 16 + (lane & 15)];
#pragma unroll
      for (int a = 0; a < TMI; ++a)
#pragma unroll
        for (int b = 0; b < TNI; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_4x4x4f64(af[a], bf[b], acc[a][b], 0, 0, 0);
    }
    if (kt + 1 < nk) {
      pa.store(As[cur ^ 1], tid);
      pb.store(Bs[cur ^ 1], tid);
    }
    __syncthreads();
  }

  double* __restrict__ Y = p.y2 + (int64_t)pair * vv;
#pragma unroll
  for (int a = 0; a < TMI; ++a)
#pragma unroll
    for (int b = 0; b < TNI; ++b) {
      const int ga = m0 + wm * WTM + a * 4 + (lane >> 4);
      const int gb = n0 + wn * WTN + b * 16 + (lane & 15);
      if (ga < v && gb < v) Y[(int64_t)ga * v + gb] = acc[a][b];
    }
}

struct OccArgs {
  int o, v, ch, nchunks;
  const double* f_oo;
  const double* f_vv;
  const double* x1;
  const double* x2;
  double* y1;
  double* y2;  // holds the virtual part on entry
};

// Singles rows of A_F (f_ov-free part): 16 outputs per workgroup (its index
// among the singles workgroups is sb), 16 lanes per output, summed by a
// fixed-order butterfly.
__device__ inline void singles_part(const OccArgs& p, int sb) {
  const int tid = threadIdx.x, o = p.o, v = p.v;
  const int64_t ov = (int64_t)o * v;
  const int w = tid >> 4, l = tid & 15;
  const int64_t out = (int64_t)sb * 16 + w;
  double part = 0.0;
  if (out < ov) {
    const int i = (int)(out / v), a = (int)(out % v);
    for (int c = l; c < v; c += 16) part += p.f_vv[(int64_t)a * v + c] * p.x1[(int64_t)i * v + c];
    for (int k = l; k < o; k += 16) part -= p.f_oo[(int64_t)k * o + i] * p.x1[(int64_t)k * v + a];
  }
  for (int m = 8; m > 0; m >>= 1) part += __shfl_xor(part, m, 16);
  if (out < ov && l == 0) p.y1[out] = part;
}

// Dynamic LDS: xs[o*o][ch] then fo[o][o].
__global__ __launch_bounds__(256) void fock_occ_kernel(OccArgs p) {
  extern __shared__ double lds[];
  const int o = p.o, v = p.v, ch = p.ch;
  const int oo = o * o;
  const int64_t vv = (int64_t)v * v;
  const int tid = threadIdx.x;

  if ((int)blockIdx.x < p.nchunks) {
    double* xs = lds;
    double* fo = lds + (int64_t)oo * ch;
    const int64_t ab0 = (int64_t)blockIdx.x * ch;
    for (int q = tid; q < oo * ch; q += 256) {
      const int pr = q / ch, e = q % ch;
      xs[q] = ab0 + e < vv ? p.x2[(int64_t)pr * vv + ab0 + e] : 0.0;
    }
    for (int q = tid; q < oo; q += 256) fo[q] = p.f_oo[q];
    __syncthreads();
    const int e = tid % ch;
    const int groups = 256 / ch;
    if (ab0 + e < vv) {
      // four pairs per round: their global loads are issued together
      constexpr int R = 4;
      for (int pr0 = tid / ch; pr0 < oo; pr0 += R * groups) {
        double yin[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int pr = pr0 + r * groups;
          const int64_t idx = (int64_t)(pr < oo ? pr : 0) * vv + ab0 + e;
          yin[r] = p.y2[idx];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int pr = pr0 + r * groups;
          if (pr >= oo) break;
          const int i = pr / o, j = pr % o;
          double occ = 0.0;
          for (int k = 0; k < o; ++k)
            occ += fo[k * o + i] * xs[(k * o + j) * ch + e] + fo[k * o + j] * xs[(i * o + k) * ch + e];
          const int64_t idx = (int64_t)pr * vv + ab0 + e;
          p.y2[idx] = yin[r] - occ;
        }
      }
    }
  } else {
    singles_part(p, blockIdx.x - p.nchunks);
  }
}

bool aligned16(const void* q) { return ((uintptr_t)q & 15u) == 0; }

void launch_vir(const FockOp& op, const double* x2, double* y2, hipStream_t s) {
  VirArgs a;
  a.v = op.v;
  a.tiles_m = (int)ceil_div(op.v, op.bm);
  a.tiles = op.tiles;
  a.units = op.tiles * op.o * op.o;
  a.per_xcd = (int)ceil_div(a.units, 8);
  a.vec = (op.v % 2 == 0 && aligned16(x2) && aligned16(op.f_vv)) ? 1 : 0;
  a.f_vv = op.f_vv;
  a.x2 = x2;
  a.y2 = y2;
  dim3 grid((unsigned)(8 * a.per_xcd));
  // contraction panels of 32 for the 32-wide blocks when that pads v no
  // more than panels of 16 (measured: the wider blocks run better with 16)
  const bool bk32 = op.bm == 32 && ceil_div(op.v, 32) * 32 <= ceil_div(op.v, 16) * 16;
  switch (op.bm * 2 + (bk32 ? 1 : 0)) {
    case 64: fock_vir_kernel<32, 2, 16><<<grid, 256, 0, s>>>(a); break;
    case 65: fock_vir_kernel<32, 2, 32><<<grid, 256, 0, s>>>(a); break;
    case 96: fock_vir_kernel<48, 4, 16><<<grid, 256, 0, s>>>(a); break;
    case 97: fock_vir_kernel<48, 4, 32><<<grid, 256, 0, s>>>(a); break;
    case 128: fock_vir_kernel<64, 2, 16><<<grid, 256, 0, s>>>(a); break;
    default: fock_vir_kernel<64, 2, 32><<<grid, 256, 0, s>>>(a); break;
  }
  PNK_CHECK_LAUNCH();
}

size_t occ_lds_bytes(int o, int ch) { return sizeof(double) * ((size_t)o * o * ch + (size_t)o * o); }

void launch_occ(const FockOp& op, const double* x1, const double* x2, double* y1, double* y2, hipStream_t s) {
  OccArgs a;
  a.o = op.o;
  a.v = op.v;
  a.ch = op.ch;
  a.nchunks = op.nchunks;
  a.f_oo = op.f_oo;
  a.f_vv = op.f_vv;
  a.x1 = x1;
  a.x2 = x2;
  a.y1 = y1;
  a.y2 = y2;
  fock_occ_kernel<<<(unsigned)op.nparts(), 256, occ_lds_bytes(op.o, op.ch), s>>>(a);
  PNK_CHECK_LAUNCH();
}

}  // namespace

// Virtual kernel: the block edge among 32 / 48 / 64 that wastes the fewest
// padded outputs (v^2 / (tiles * bm^2)); among near-ties the largest edge
// that still gives at least 512 workgroups (two per CU), else the smallest.
// Occupied kernel: the widest chunk (64 .. 16 elements, 8 only when 16 does
// not fit) whose LDS stays within 64 KB (two workgroups per CU) and that
// still gives 512 workgroups.
bool fock_op_plan(FockOp& op) {
  if (op.o < 1 || op.v < 1 || op.o > kFockOpMaxOcc) return false;
  const int cand[3] = {32, 48, 64};
  double util[3], best = 0.0;
  for (int c = 0; c < 3; ++c) {
    const double t = (double)ceil_div(op.v, cand[c]) * cand[c];
    util[c] = (double)op.v * op.v / (t * t);
    best = std::max(best, util[c]);
  }
  int pick = -1;
  for (int c = 2; c >= 0; --c) {
    if (util[c] < 0.98 * best) continue;
    const int64_t tiles = ceil_div(op.v, cand[c]) * ceil_div(op.v, cand[c]);
    if ((int64_t)op.o * op.o * tiles >= 512) { pick = c; break; }
  }
  if (pick < 0)
    for (int c = 0; c < 3; ++c)
      if (util[c] >= 0.98 * best) { pick = c; break; }
  op.bm = cand[pick];
  const int64_t tm = ceil_div(op.v, op.bm);
  op.tiles = (int)(tm * tm);

  const int64_t vv = (int64_t)op.v * op.v;
  // (at least 16 elements: a full 128-byte line per pair and chunk)
  op.ch = 0;
  for (int ch : {64, 32, 16, 8}) {
    if (occ_lds_bytes(op.o, ch) > 64 * 1024) continue;
    if (op.ch == 0) op.ch = ch;  // widest that fits, whatever the count
    if (ceil_div(vv, ch) >= 512 || ch == 16) { op.ch = ch; break; }
  }
  if (op.ch == 0) return false;
  op.nchunks = (int)ceil_div(vv, op.ch);
  op.nsingles = (int)ceil_div((int64_t)op.o * op.v, 16);
  return (int64_t)op.tiles * op.o * op.o < (1ll << 31) - 8 && op.nparts() <= 0x7fffffff;
}

void fock_op_apply(const FockOp& op, const double* x1, const double* x2, double* y1, double* y2, hipStream_t s) {
  PNK_REQUIRE(op.bm > 0, "fock_op: not planned");
  PNK_REQUIRE(x1 != y1 && x2 != y2, "fock_op: output must not alias the input");
  launch_vir(op, x2, y2, s);
  launch_occ(op, x1, x2, y1, y2, s);
}

}  // namespace pnk
