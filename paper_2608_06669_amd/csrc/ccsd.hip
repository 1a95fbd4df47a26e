// CCSD residual / Jacobian-vector product / Fock operator as a sequence of
// matrix-core contractions (see ccsd.hpp).
//
// Index names follow the paper: i,j,k,l occupied; a,b,c,d virtual. Layouts:
// t1[i][a], t2[i][j][a][b], DF blocks X[P][p][q] with P < naux and an extra
// slice P = naux holding the one-electron operator h, dressed like L.
//
// Working equations (T1-dressed closed-shell CCSD; the CCD part is the
// paper's Appendix A with the g_c^a and K signs read as in its
// random-gauge form):
//   r_i^a   = F~_ai + sum_kcd (ac|kd)~ u_ik^cd - sum_klc (ki|lc)~ u_kl^ac
//             + sum_kc F~_kc u_ik^ac
//   r_ij^ab = (ai|bj)~ + sum_cd (ac|bd)~ t_ij^cd + sum_kl W_klij t_kl^ab
//             + P_ij^ab [ sum_c Gv_bc t_ij^ac - sum_k Go_kj t_ik^ab
//                         + sum_kc J_ai,kc u_jk^bc - sum_kc K_ki,ac t_kj^cb
//                         - sum_kc K_ki,bc t_kj^ac ]
// with u = 2 t_ij^ab - t_ij^ba, W_klij = (ki|lj)~ + sum_cd (kc|ld) t_ij^cd,
// Gv_bc = F~_bc - sum (kc|ld) u_kl^bd, Go_kj = F~_kj + sum (kc|ld) u_jl^cd,
// J_ai,kc = (ai|kc)~ + 1/2 sum (kc|ld) u_il^ad - 1/2 sum (kd|lc) t_il^ad,
// K_ki,ac = (ki|ac)~ - 1/2 sum (kd|lc) t_il^da, P_ij^ab Z = Z_ij^ab + Z_ji^ba.
// The dressed ladder splits as sum_cd (ac|bd) t_ij^cd (precomputed
// W_vvvv) + P_ij^ab[-sum_k t_k^a Z'_ij,kb], Z' = Z - 1/2 Y t1 with
// Z_ij,kb = sum_cd (kc|bd) t_ij^cd and Y_ij,kl = sum_cd (kc|ld) t_ij^cd.

#include "ccsd.hpp"
#include "fock_op.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstdio>
#include <cstring>

#include "cc_kernels.hpp"
#include "eig.hpp"
#include "gemm.hpp"
#include "tensor_ops.hpp"

namespace pnk {

// ------------------------------------------------------------- arena ----

namespace {
void release(void* p, hipStream_t s, bool async) {
  if (!p) return;
  if (async) (void)hipFreeAsync(p, s);
  else (void)hipFree(p);
}
}  // namespace

Arena::~Arena() { release(base_, stream_, async_); }

void Arena::reserve(size_t bytes, hipStream_t stream, bool stream_ordered) {
  release(base_, stream_, async_);
  base_ = nullptr;
  cap_ = used_ = 0;
  stream_ = stream;
  async_ = stream_ordered;
  if (bytes == 0) return;
  hipError_t e = stream_ordered ? hipMallocAsync((void**)&base_, bytes, stream) : hipMalloc(&base_, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    base_ = nullptr;
    throw OomError("device allocation of " + std::to_string(bytes) + " bytes failed");
  }
  cap_ = bytes;
}

void* Arena::take_bytes(size_t bytes) {
  const size_t a = (used_ + 255) & ~size_t(255);
  if (a + bytes > cap_) throw OomError("engine arena exhausted");
  used_ = a + bytes;
  return base_ + a;
}

// ------------------------------------------------------------ timers ----

Timers::~Timers() {
  reset();
  for (auto& p : pool_) { (void)hipEventDestroy(p.a); (void)hipEventDestroy(p.b); }
}

void Timers::begin(int slot, hipStream_t s) {
  Pair p;
  if (pool_.empty()) {
    PNK_HIP(hipEventCreate(&p.a));
    PNK_HIP(hipEventCreate(&p.b));
  } else {
    p = pool_.back();
    pool_.pop_back();
  }
  p.slot = slot;
  PNK_HIP(hipEventRecord(p.a, s));
  used_.push_back(p);
  is_open_[slot] = true;
}

void Timers::end(int slot, hipStream_t s) {
  for (auto it = used_.rbegin(); it != used_.rend(); ++it)
    if (it->slot == slot) {
      PNK_HIP(hipEventRecord(it->b, s));
      break;
    }
  is_open_[slot] = false;
}

void Timers::read(int slot, int* count, double* total_ms) {
  for (auto& p : used_) {
    PNK_HIP(hipEventSynchronize(p.b));
    float ms = 0.f;
    PNK_HIP(hipEventElapsedTime(&ms, p.a, p.b));
    count_[p.slot] += 1;
    total_[p.slot] += ms;
    pool_.push_back(p);
  }
  used_.clear();
  *count = count_[slot];
  *total_ms = total_[slot];
}

void Timers::reset() {
  for (auto& p : used_) {
    (void)hipEventSynchronize(p.b);
    pool_.push_back(p);
  }
  used_.clear();
  for (int k = 0; k < kTimerSlots; ++k) { count_[k] = 0; total_[k] = 0.0; is_open_[k] = false; }
}

// ----------------------------------------------------------- sizing -----

namespace {

// n rounded up to a multiple of m
int64_t pad_to(int64_t n, int64_t m) { return (n + m - 1) / m * m; }

struct Sizes {
  int64_t o, v, naux, np, n, ov, n2, p2, p2m, o2, o2m, wna;
  int64_t p2k, p2mk, ldp, ldm, o2k, o2mk;  // padded lengths (LadderLayout)
  explicit Sizes(int o_, int v_, int naux_)
      : o(o_), v(v_), naux(naux_), np(naux_ + 1), n(o_ + v_), ov((int64_t)o_ * v_), n2(ov * ov),
        p2((int64_t)v_ * (v_ + 1) / 2), p2m((int64_t)v_ * (v_ - 1) / 2), o2((int64_t)o_ * (o_ + 1) / 2),
        o2m((int64_t)o_ * (o_ - 1) / 2), p2k(pad_to(p2, 8)), p2mk(pad_to(p2m, 8)), ldp(pad_to(p2 + ov + o2, 8)),
        ldm(p2m ? pad_to(p2m + ov + o2m, 8) : 0), o2k(pad_to(o2, 2)), o2mk(pad_to(o2m, 2)) {
    // (ac|bd) is built for blocks of `wna` values of a at a time
    const int64_t v3 = v * v * v;
    wna = std::max<int64_t>(1, std::min<int64_t>(v, (32ll << 20) / v3));
  }
};

// Split-K scratch. Products with few output tiles, or whose last tiles would
// leave the chip idle, cut them along k; the chunk count is also capped by
// this size. 16 times the largest o^2 v^2-class tensor, at most 16 M elements
// (128 MB): room for eight chunks of the last 177 tiles of the ladder at o =
// 20, v = 180.
int64_t splitk_elems(const Sizes& z) {
  const int64_t big = std::max<int64_t>({z.o * z.o * z.v * z.v, z.ov * z.ov, (int64_t)z.o * z.o * z.o * z.o});
  return std::min<int64_t>(std::max<int64_t>(16 * big, 1 << 16), 16 * 1024 * 1024);
}

// Rounded copies of FP64 operands for the FP32/BF16 products of J v: room
// for both operands of the largest dual product (the ring term, 2ov x 2ov),
// with rows padded to 16 bytes.
int64_t cast_bytes(const Sizes& z, const EngineOptions& opt) {
  if (!opt.lowp_f32 && !opt.lowp_bf16) return 0;
  // (rows of the packed copies are padded along k, to 64 elements in BF16)
  return (opt.lowp_f32 ? 4 : 2) * (4 * z.n2 + 160 * z.ov) + (1 << 20);
}

// Calls `f(count_doubles)` for every FP64 buffer in allocation order, and
// `g(count_bytes)` for the low-precision copies.
template <class F, class G>
void for_each_buffer(const Sizes& z, const EngineOptions& opt, F f, G g) {
  const int64_t o = z.o, v = z.v, naux = z.naux, np = z.np, n = z.n, ov = z.ov, n2 = z.n2;
  // constants
  f(o * o); f(ov); f(v * v); f(n * n); f(n * n); f(naux); f(naux * o * n);
  f(np * o * o); f(np * ov); f(np * ov); f(np * v * v);
  const int64_t p2 = z.p2, p2m = z.p2m;
  f(z.p2k * z.ldp); f(z.p2mk * z.ldm); f(z.wna * v * v * v); g(4 * p2); g(4 * p2); g(4 * p2m); g(4 * p2m);
  for (int k = 0; k < 4; ++k) f(n2);
  if (opt.lowp_f32) {
    g(4 * p2 * pad_to(p2, 4)); g(4 * p2m * pad_to(p2m, 4));
    g(4 * o * v * v * v); g(4 * n2); g(4 * n2); g(4 * n2); g(4 * n2);
  }
  if (opt.lowp_bf16) {
    g(2 * p2 * pad_to(p2, 64)); g(2 * p2m * pad_to(p2m, 64));
    g(2 * ov * pad_to(v * v, 64)); g(2 * n2); g(2 * ov * pad_to(ov, 64)); g(2 * ov * pad_to(ov, 64)); g(2 * n2);
  }
  g(cast_bytes(z, opt));
  // intermediates, value and tangent
  for (int rep = 0; rep < 2; ++rep) {
    f(np * o * o); f(np * ov); f(np * v * v); f(naux); f(naux * o * o);
    f(o * o); f(ov); f(v * v);
    f(n2); f(n2);  // Tsia, Uia
    f(v * v); f(o * o); f(o * o * o * o); f(o * o * ov);
    f(n2); f(n2);                       // M, K
    f(naux * ov); f(o * o * ov);  // QT, Kilc
    f(z.o2k * z.p2k); f(z.o2mk * z.p2mk);  // Tp, Tm
    if (rep == 0) {  // Tmp, X, Kilj, Q, Rp, Rm
      f(n2); f(n2); f(o * o * o * o); f(naux * ov); f(z.o2 * z.ldp); f(z.o2m * z.ldm);
    }
    if (rep == 0 || o == 1 || !(opt.lowp_f32 || opt.lowp_bf16)) { f(z.o2 * z.o2k); f(z.o2m * z.o2mk); }  // Wp, Wm
    if (opt.lowp_f32 || opt.lowp_bf16) {  // Tia, U, Uklca, Uail, J, KilcT, Wkl
      for (int k = 0; k < 5 - 2 * rep; ++k) f(n2);
      f(o * o * ov); f(o * o * o * o);
    }
  }
  f(reduce_partials_size(64));
  f(ov + n2);  // zeros
  f(splitk_elems(z));
  f(ov + n2); f(ov + n2);  // graph tangent in / out
}

}  // namespace

size_t engine_bytes(int o, int v, int naux, const EngineOptions& opt) {
  Sizes z(o, v, naux);
  size_t total = 0;
  auto add = [&](int64_t bytes) { total += ((size_t)bytes + 255) & ~size_t(255); };
  for_each_buffer(z, opt, [&](int64_t nd) { add(nd * 8); }, [&](int64_t nb) { add(nb); });
  return total + 256;
}

// ----------------------------------------------------------- engine -----

Engine::Engine(int o, int v, int naux, const EngineOptions& opt)
    : o_(o), v_(v), naux_(naux), np_(naux + 1), ov_((int64_t)o * v), n2_((int64_t)o * v * o * v), opt_(opt) {
  PNK_REQUIRE(o > 0 && v > 0 && naux > 0, "nocc, nvir and naux must be positive");
  Sizes z(o, v, naux);
  arena_.reserve(engine_bytes(o, v, naux, opt), opt.alloc_stream, opt.stream_ordered);
  const int64_t O = o, V = v, NA = naux, NP = np_, N = o + v, OV = ov_, N2 = n2_;
  auto take = [&](int64_t n) { return arena_.take<double>((size_t)n); };
  f_oo_ = take(O * O); f_ov_ = take(OV); f_vv_ = take(V * V); fock_ = take(N * N); h_ = take(N * N); dtr_ = take(NA);
  Lo_ = take(NA * O * N);
  Loo0.v = take(NP * O * O); Lov0.v = take(NP * OV); Lvo0.v = take(NP * OV); Lvv0.v = take(NP * V * V);
  lad_ = {z.p2, z.p2m, z.o2, z.o2m, z.p2k, z.p2mk, z.ldp, z.ldm, z.o2k, z.o2mk};
  wblk_na_ = (int)z.wna;
  S.v = take(z.p2k * z.ldp); Am.v = take(z.p2mk * z.ldm); wblk_ = take(z.wna * V * V * V);
  pair_a_ = arena_.take<int>(z.p2); pair_b_ = arena_.take<int>(z.p2);
  mpair_a_ = arena_.take<int>(z.p2m); mpair_b_ = arena_.take<int>(z.p2m);
  Iovov.v = take(N2); Ix.v = take(N2); Lh.v = take(N2); Itil.v = take(N2);
  // the low-precision ladder tensors keep rows of a 16-byte multiple (the
  // pair counts v(v+1)/2, v(v-1)/2 need not be), for vector loads
  ld32_ = pad_to(z.p2, 4); ld32m_ = pad_to(z.p2m, 4);
  ld16_ = pad_to(z.p2, 64); ld16m_ = pad_to(z.p2m, 64);  // whole 64-deep panels, zero-padded
  if (opt.lowp_f32) {
    S.lp32 = arena_.take<float>(z.p2 * ld32_); Am.lp32 = arena_.take<float>(z.p2m * ld32m_);
    Wov.lp32 = arena_.take<float>(O * V * V * V);
    Ioovv.lp32 = arena_.take<float>(N2); Iovov.lp32 = arena_.take<float>(N2);
    Ix.lp32 = arena_.take<float>(N2); Ikldc.lp32 = arena_.take<float>(N2);
  }
  if (opt.lowp_bf16) {
    S.lp16 = arena_.take<uint16_t>(z.p2 * ld16_); Am.lp16 = arena_.take<uint16_t>(z.p2m * ld16m_);
    ldw16_ = pad_to(V * V, 64);  // rows along k, zero-padded to whole panels
    Wov.lp16 = arena_.take<uint16_t>(OV * ldw16_);
    // the ring integrals in BF16 are read along k (the matrix-core operand
    // layout), rows zero-padded to whole 64-deep panels: Iovov as is (it is
    // symmetric), Ix transposed
    ldov16_ = pad_to(OV, 64);
    Ioovv.lp16 = arena_.take<uint16_t>(N2); Iovov.lp16 = arena_.take<uint16_t>(OV * ldov16_);
    Ix.lp16 = arena_.take<uint16_t>(OV * ldov16_); Ikldc.lp16 = arena_.take<uint16_t>(N2);
  }
  cast_bytes_ = cast_bytes(z, opt);
  if (cast_bytes_) cast_ws_ = arena_.take<char>((size_t)cast_bytes_);
  Ten* inter[] = {&Loo, &Lvo, &Lvv, &this->D, &LooT, &Foo, &Fov, &Fvv,
                  &Tsia, &Uia, &Tmp, &X,
                  &Gv, &Go, &Kilj, &Y, &Z, &M, &K, &Q, &QT, &Kilc,
                  &Tp, &Tm, &Rp, &Rm, &Wp, &Wm,
                  &Tia, &U, &Uklca, &Uail, &J, &KilcT, &Wkl};
  const int64_t isz[] = {NP * O * O, NP * OV, NP * V * V, NA, NA * O * O, O * O, OV, V * V,
                         N2, N2, N2, N2,
                         V * V, O * O, O * O * O * O, O * O * O * O, O * O * OV, N2, N2,
                         NA * OV, NA * OV, O * O * OV,
                         z.o2k * z.p2k, z.o2mk * z.p2mk, z.o2 * z.ldp, z.o2m * z.ldm, z.o2 * z.o2k, z.o2m * z.o2mk,
                         N2, N2, N2, N2, N2, O * O * OV, O * O * O * O};
  const size_t nlow = opt.lowp_f32 || opt.lowp_bf16 ? 0 : 7;  // the last seven: FP32 / BF16 only
  static_assert(sizeof(inter) / sizeof(inter[0]) == sizeof(isz) / sizeof(isz[0]), "buffer table");
  // read only in the pass that writes them: one array for value and tangent
  Ten* scratch[] = {&Tmp, &X, &Kilj, &Q, &Rp, &Rm};
  for (int rep = 0; rep < 2; ++rep)
    for (size_t k = 0; k + nlow < sizeof(isz) / sizeof(isz[0]); ++k) {
      Ten* t = inter[k];
      t->var = true;
      if (rep == 0) t->v = take(isz[k]);
      else if (std::find(std::begin(scratch), std::end(scratch), t) != std::end(scratch)) t->d = t->v;
      else if (t != &J && t != &Uail && (nlow != 0 || o == 1 || (t != &Wp && t != &Wm))) t->d = take(isz[k]);
    }
  // An FP64 tangent has M, Wp and Wm, one in FP32 or BF16 J and Wkl (o^4 >=
  // o2 o2k + o2m o2mk from two occupied orbitals on)
  J.d = M.d;
  Uail.d = Tmp.d;  // (read before Tmp is first written)
  if (!nlow && o > 1) {
    Wp.d = Wkl.d;
    Wm.d = Wkl.d + z.o2 * z.o2k;
  }
  Ioovv.v = X.v;  // (prepare only: products read its copies)
  partials_ = take(reduce_partials_size(64));
  zeros_ = take(OV + N2);
  ws_elems_ = splitk_elems(z);
  ws_ = take(ws_elems_);
  tin_ = take(OV + N2);
  tout_ = take(OV + N2);
  T1.var = T2.var = R1.var = R2.var = true;
  fop_.o = o;
  fop_.v = v;
  fop_.f_oo = f_oo_;
  fop_.f_vv = f_vv_;
  fop_ok_ = fock_op_plan(fop_);
  (void)z;
}

Engine::~Engine() {
  for (GraphSlot* g : {&res_slot_, &jvp_slot_[0], &jvp_slot_[1], &jvp_slot_[2]})
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (cap_) (void)hipStreamDestroy(cap_);
}

// Record run(m) on a private stream (stream capture does not execute) and
// instantiate it. Returns false (and leaves the slot empty) if the runtime
// refuses; the caller then runs eagerly.
bool Engine::capture(Mode m, GraphSlot* slot) {
  if (!cap_ && hipStreamCreateWithFlags(&cap_, hipStreamNonBlocking) != hipSuccess) {
    (void)hipGetLastError();
    cap_ = nullptr;
    return false;
  }
  hipStream_t saved = s_;
  Timers* tm = timers_;
  timers_ = nullptr;
  s_ = cap_;
  hipGraph_t g = nullptr;
  bool ok = false;
  if (hipStreamBeginCapture(cap_, hipStreamCaptureModeThreadLocal) == hipSuccess) {
    // a failure while recording must not leave a partial graph behind
    bool threw = false;
    try {
      run(m);
    } catch (const std::exception& e) {
      threw = true;
      if (std::getenv("PNK_DEBUG")) std::fprintf(stderr, "pnk: graph capture failed: %s\n", e.what());
    }
    if (hipStreamEndCapture(cap_, &g) == hipSuccess && g && !threw &&
        hipGraphInstantiate(&slot->exec, g, nullptr, nullptr, 0) == hipSuccess)
      ok = true;
  }
  if (g) (void)hipGraphDestroy(g);
  (void)hipGetLastError();
  if (!ok) slot->exec = nullptr;
  s_ = saved;
  timers_ = tm;
  mode_ = Mode::Value;
  return ok;
}

// True when slot holds a graph for these buffers. A graph is recorded on the
// second consecutive call with the same key (so one-off evaluations, such as
// the residual at t = 0, stay eager).
bool Engine::graph_ready(GraphSlot* slot, const void* k0, const void* k1, const void* k2, const void* k3, Mode m) {
  if (!use_graphs_) return false;
  const bool same = slot->key[0] == k0 && slot->key[1] == k1 && slot->key[2] == k2 && slot->key[3] == k3;
  if (same && slot->exec) return true;
  if (!same) {
    if (slot->exec) (void)hipGraphExecDestroy(slot->exec);
    slot->exec = nullptr;
    slot->key[0] = k0; slot->key[1] = k1; slot->key[2] = k2; slot->key[3] = k3;
    slot->hits = 1;
    return false;
  }
  if (++slot->hits < 2) return false;
  return capture(m, slot);
}

// ---------------------------------------------------- op primitives -----

namespace {
GemmDesc gd(int M, int N, int K, int64_t am, int64_t ak, int64_t bk, int64_t bn, int64_t cm, int64_t cn,
            double alpha = 1.0, double beta = 0.0) {
  GemmDesc d;
  d.M = M; d.N = N; d.K = K;
  d.a_m = am; d.a_k = ak; d.b_k = bk; d.b_n = bn; d.c_m = cm; d.c_n = cn;
  d.alpha = alpha; d.beta = beta;
  return d;
}
GemmDesc batch0(GemmDesc d, int nb, int64_t ab, int64_t bb, int64_t cb) {
  d.nb0 = nb; d.a_b0 = ab; d.b_b0 = bb; d.c_b0 = cb;
  return d;
}
}  // namespace

void Engine::operand(const Ten& t, bool tangent, const void** p, Prec* prec) const {
  if (tangent) { *p = t.d; *prec = Prec::F64; return; }
  if (mode_ == Mode::Tangent && !t.var) {
    if (jprec_ == Prec::BF16 && t.lp16) { *p = t.lp16; *prec = Prec::BF16; return; }
    if (jprec_ == Prec::F32 && t.lp32) { *p = t.lp32; *prec = Prec::F32; return; }
  }
  *p = t.v;
  *prec = Prec::F64;
}

// C = alpha A B + beta C, or its tangent dC = alpha (dA B + A dB) + beta dC;
// with src, alpha A B + beta src
void Engine::mm(const GemmDesc& d, const Ten& A, const Ten& B, const Ten& C, const Ten* src, int64_t off,
                double beta) {
  const double f = 2.0 * d.M * d.N * d.K * (double)d.nb0 * d.nb1;
  GemmDesc e = with_ws(d);
  if (src) {
    const bool there = mode_ == Mode::Value || src->var;  // (the tangent of a constant is zero)
    e.beta = there ? beta : 0.0;
    e.Cin = there ? out(*src) + off : nullptr;
  }
  if (mode_ == Mode::Value) {
    mm_flops_ += f;
    gemm64(e, A.v, B.v, C.v, s_);
    return;
  }
  // the tangent of a product with one varying operand is one product, with
  // two varying operands two
  mm_flops_ += (A.var && B.var) ? 2.0 * f : f;
  PNK_REQUIRE(A.var || B.var, "internal: variable output of a constant product");
  const void *pa, *pb;
  Prec qa, qb;
  if (A.var && B.var) {
    // dA B + A dB as one launch when the operand precisions agree
    const void *pa2, *pb2;
    Prec qa2, qb2;
    operand(A, true, &pa, &qa);
    operand(B, false, &pb, &qb);
    operand(A, false, &pa2, &qa2);
    operand(B, true, &pb2, &qb2);
    if (qa == qa2 && qb == qb2) {
      gemm_sum(e, pa, pb, pa2, pb2, qa, qb, C.d, Prec::F64, jprec_, s_);
      return;
    }
  }
  bool first = true;
  if (A.var) {
    operand(A, true, &pa, &qa);
    operand(B, false, &pb, &qb);
    gemm(e, pa, qa, pb, qb, C.d, Prec::F64, jprec_, s_);
    first = false;
  }
  if (B.var) {
    if (!first) {
      e.beta = 1.0;
      e.Cin = nullptr;
    }
    operand(A, false, &pa, &qa);
    operand(B, true, &pb, &qb);
    gemm(e, pa, qa, pb, qb, C.d, Prec::F64, jprec_, s_);
  }
}

// (in, out and src depend on the amplitudes)
void Engine::perm(const Ten& in, const Ten& to, int d0, int d1, int d2, int d3, int p0, int p1, int p2, int p3,
                  double alpha, double beta, const Ten* src) {
  const int dims[4] = {d0, d1, d2, d3};
  const int pm[4] = {p0, p1, p2, p3};
  permute4(out(in), out(to), dims, pm, alpha, beta, s_, src ? out(*src) : nullptr);
}

// ------------------------------------------------------------ prepare ---

void Engine::fetch_fock(std::vector<double>* foo, std::vector<double>* fvv, hipStream_t s) const {
  foo->resize((size_t)o_ * o_);
  fvv->resize((size_t)v_ * v_);
  PNK_HIP(hipMemcpyAsync(foo->data(), f_oo_, foo->size() * sizeof(double), hipMemcpyDeviceToHost, s));
  PNK_HIP(hipMemcpyAsync(fvv->data(), f_vv_, fvv->size() * sizeof(double), hipMemcpyDeviceToHost, s));
  PNK_HIP(hipStreamSynchronize(s));
}

// Into fock_ and h_, which are free once the blocks are extracted: [eps_o |
// eps_v | ut_o | ut_v] (o + v + o^2 + v^2 <= (o + v)^2 doubles) and u_o
void Engine::compute_eigen(const std::vector<double>& foo, const std::vector<double>& fvv, hipStream_t s) {
  const size_t o = o_, v = v_;
  std::vector<double> buf(o + v + o * o + v * v);
  double *eo = buf.data(), *ev = eo + o, *uo = ev + v, *uv = uo + o * o;
  bool diag_o = false, diag_v = false;
  eigen_ok_ = symmetric_eigen(foo.data(), o_, eo, uo, &diag_o) && symmetric_eigen(fvv.data(), v_, ev, uv, &diag_v);
  eigen_done_ = true;
  if (!eigen_ok_) return;
  PNK_HIP(hipMemcpyAsync(fock_, buf.data(), buf.size() * sizeof(double), hipMemcpyHostToDevice, s));
  PNK_HIP(hipStreamSynchronize(s));  // buf goes out of scope
  eigen_.o = o_;
  eigen_.v = v_;
  eigen_.eps_o = fock_;
  eigen_.eps_v = fock_ + o;
  eigen_.ut_o = eigen_.u_o = nullptr;
  if (!diag_o) {
    std::vector<double> u(o * o);
    for (size_t i = 0; i < o; ++i)
      for (size_t k = 0; k < o; ++k) u[i * o + k] = uo[k * o + i];
    PNK_HIP(hipMemcpyAsync(h_, u.data(), u.size() * sizeof(double), hipMemcpyHostToDevice, s));
    PNK_HIP(hipStreamSynchronize(s));
    eigen_.ut_o = fock_ + o + v;
    eigen_.u_o = h_;
  }
  eigen_.ut_v = diag_v ? nullptr : fock_ + o + v + o * o;
}

const FockEigen* Engine::fock_eigen(hipStream_t s) {
  if (!eigen_done_) {
    std::vector<double> foo, fvv;
    fetch_fock(&foo, &fvv, s);
    compute_eigen(foo, fvv, s);
  }
  return eigen_ok_ ? &eigen_ : nullptr;
}

void Engine::prepare(const ProblemView& p, hipStream_t s, bool with_eigen) {
  PNK_REQUIRE(p.o == o_ && p.v == v_ && p.naux == naux_, "prepare: dimensions differ from the engine's");
  s_ = s;
  mode_ = Mode::Value;
  const int o = o_, v = v_, naux = naux_, n = o + v;
  const int64_t ov = ov_, vv = (int64_t)v * v;
  PNK_HIP(hipMemcpyAsync(f_oo_, p.f_oo, sizeof(double) * o * o, hipMemcpyDeviceToDevice, s));
  PNK_HIP(hipMemcpyAsync(f_ov_, p.f_ov, sizeof(double) * ov, hipMemcpyDeviceToDevice, s));
  PNK_HIP(hipMemcpyAsync(f_vv_, p.f_vv, sizeof(double) * vv, hipMemcpyDeviceToDevice, s));
  eigen_done_ = false;
  std::vector<double> foo, fvv;
  if (with_eigen) fetch_fock(&foo, &fvv, s);
  // h = f - G[L], G[L]_pq = sum_P 2 L_pq d_P - sum_Pk L_pk L_kq
  assemble_fock(o, v, f_oo_, f_ov_, f_vv_, fock_, s);
  copy((int64_t)n * n, fock_, h_, s);
  trace_occ(naux, o, n, p.L, dtr_, s);
  gemm64(with_ws(gd(1, n * n, naux, 0, 1, (int64_t)n * n, 1, 0, 1, -2.0, 1.0)), dtr_, p.L, h_, s);
  extract_occ_rows(naux, o, n, p.L, Lo_, s);
  gemm64(with_ws(gd(n, n, naux * o, 1, n, n, 1, n, 1, 1.0, 1.0)), Lo_, Lo_, h_, s);
  extract_blocks(naux, o, v, p.L, h_, Loo0.v, Lov0.v, Lvo0.v, Lvv0.v, s);
  const int64_t p2 = lad_.p2, p2m = lad_.p2m, ldp = lad_.ldp, ldm = lad_.ldm;
  // zero padding the products run over
  fill(lad_.p2k * ldp - p2 * ldp, 0.0, S.v + p2 * ldp, s);
  fill(lad_.p2mk * ldm - p2m * ldm, 0.0, Am.v + p2m * ldm, s);
  for (Ten* t : {&Tp, &Tm}) {
    const bool sym = t == &Tp;
    const int64_t row = sym ? lad_.p2k : lad_.p2mk, r0 = sym ? lad_.o2 : lad_.o2m, r1 = sym ? lad_.o2k : lad_.o2mk;
    fill((r1 - r0) * row, 0.0, t->v + r0 * row, s);
    fill((r1 - r0) * row, 0.0, t->d + r0 * row, s);
  }
  // symmetry-adapted (ac|bd): pair tables, then blocks of a at a time:
  // Wblk[a - a0][b][c][d] = sum_P L_ac L_bd (batch b0 = b, b1 = a - a0),
  // packed into S (a <= b, c <= d; rows a = b halved) and A (a < b, c < d)
  {
    std::vector<int> pa(p2), pb(p2), ma(std::max<int64_t>(p2m, 1)), mb(std::max<int64_t>(p2m, 1));
    int64_t k = 0, km = 0;
    for (int a = 0; a < v; ++a)
      for (int b = a; b < v; ++b) {
        pa[k] = a; pb[k] = b; ++k;
        if (b > a) { ma[km] = a; mb[km] = b; ++km; }
      }
    PNK_HIP(hipMemcpyAsync(pair_a_, pa.data(), p2 * sizeof(int), hipMemcpyHostToDevice, s));
    PNK_HIP(hipMemcpyAsync(pair_b_, pb.data(), p2 * sizeof(int), hipMemcpyHostToDevice, s));
    if (p2m > 0) {
      PNK_HIP(hipMemcpyAsync(mpair_a_, ma.data(), p2m * sizeof(int), hipMemcpyHostToDevice, s));
      PNK_HIP(hipMemcpyAsync(mpair_b_, mb.data(), p2m * sizeof(int), hipMemcpyHostToDevice, s));
    }
    PNK_HIP(hipStreamSynchronize(s));  // host tables go out of scope
    for (int a0 = 0; a0 < v; a0 += wblk_na_) {
      const int na = std::min(wblk_na_, v - a0);
      GemmDesc d = gd(v, v, naux, 1, vv, vv, 1, v, 1);
      d.nb0 = v; d.nb1 = na;
      d.a_b0 = 0; d.a_b1 = v;
      d.b_b0 = v; d.b_b1 = 0;
      d.c_b0 = vv; d.c_b1 = vv * v;
      gemm64(with_ws(d), Lvv0.v + (int64_t)a0 * v, Lvv0.v, wblk_, s);
      ppl_pack_w(v, a0, na, wblk_, pair_a_, pair_b_, mpair_a_, mpair_b_, S.v, ldp, Am.v, ldm, s);
    }
  }
  // further columns: (kc|bd) +- (kd|bc), blocks of k at a time through
  // Wblk[k - k0][b][c][d] = (kc|bd)
  for (int k0 = 0; k0 < o; k0 += wblk_na_) {
    const int nk = std::min(wblk_na_, o - k0);
    GemmDesc d = gd(v, v, naux, 1, ov, vv, 1, v, 1);
    d.nb0 = v; d.nb1 = nk;
    d.a_b0 = 0; d.a_b1 = v;
    d.b_b0 = v; d.b_b1 = 0;
    d.c_b0 = vv; d.c_b1 = vv * v;
    gemm64(with_ws(d), Lov0.v + (int64_t)k0 * v, Lvv0.v, wblk_, s);
    const int64_t r0 = (int64_t)k0 * v, nr = (int64_t)nk * v;
    ladder_columns(v, nr, 0, wblk_, pair_a_, pair_b_, mpair_a_, mpair_b_, S.v + p2 + r0, ldp, Am.v + p2m + r0, ldm, s);
    if (Wov.lp32) cast_f64_to_f32(nr * vv, wblk_, (float*)Wov.lp32 + r0 * vv, s);
    if (Wov.lp16) cast_f64_to_bf16_rows(nr, vv, ldw16_, wblk_, vv, (uint16_t*)Wov.lp16 + r0 * ldw16_, s);
  }
  // Ioovv[k][l][c][d] = (kc|ld)
  {
    GemmDesc d = gd(v, v, naux, 1, ov, ov, 1, v, 1);
    d.nb0 = o; d.nb1 = o;
    d.a_b0 = 0; d.a_b1 = v;
    d.b_b0 = v; d.b_b1 = 0;
    d.c_b0 = vv; d.c_b1 = vv * o;
    gemm64(with_ws(d), Lov0.v, Lov0.v, Ioovv.v, s);
  }
  // the last columns: (kc|ld) +- (kd|lc), k <= l
  ladder_columns(v, (int64_t)o * o, o, Ioovv.v, pair_a_, pair_b_, mpair_a_, mpair_b_, S.v + p2 + ov, ldp,
                 Am.v + p2m + ov, ldm, s);
  fill_columns(p2, S.v + p2 + ov + lad_.o2, ldp, ldp - (p2 + ov + lad_.o2), s);
  if (p2m > 0) fill_columns(p2m, Am.v + p2m + ov + lad_.o2m, ldm, ldm - (p2m + ov + lad_.o2m), s);
  // Iovov[(k,c)][(l,d)] = (kc|ld); Ix[l][d][k][c] = (kd|lc)
  gemm64(with_ws(gd((int)ov, (int)ov, naux, 1, ov, ov, 1, ov, 1)), Lov0.v, Lov0.v, Iovov.v, s);
  {
    const int dims[4] = {o, v, o, v};
    const int pm[4] = {2, 1, 0, 3};
    permute4(Iovov.v, Ix.v, dims, pm, 1.0, 0.0, s);
    permute4(Iovov.v, Lh.v, dims, pm, -0.5, 1.0, s, Iovov.v);  // (kc|ld) - (kd|lc) / 2
    const int dims2[4] = {o, o, v, v};
    const int pm2[4] = {0, 1, 3, 2};
    permute4(Ioovv.v, Itil.v, dims2, pm2, -1.0, 2.0, s, Ioovv.v);
    if (Ikldc.lp32 || Ikldc.lp16) {  // (kc|ld) as [k][l][d][c], staged in Tmp
      permute4(Ioovv.v, Tmp.v, dims2, pm2, 1.0, 0.0, s);
      if (Ikldc.lp32) cast_f64_to_f32(n2_, Tmp.v, (float*)Ikldc.lp32, s);
      if (Ikldc.lp16) cast_f64_to_bf16(n2_, Tmp.v, (uint16_t*)Ikldc.lp16, s);
    }
  }
  // the ladder tensors with padded rows, the others flat
  if (S.lp32) cast_f64_to_f32_rows(p2, p2, ld32_, S.v, ldp, (float*)S.lp32, s, pair_a_, pair_b_);
  if (S.lp16) cast_f64_to_bf16_rows(p2, p2, ld16_, S.v, ldp, (uint16_t*)S.lp16, s, pair_a_, pair_b_);
  if (Am.lp32) cast_f64_to_f32_rows(p2m, p2m, ld32m_, Am.v, ldm, (float*)Am.lp32, s);
  if (Am.lp16) cast_f64_to_bf16_rows(p2m, p2m, ld16m_, Am.v, ldm, (uint16_t*)Am.lp16, s);
  if (Ioovv.lp32) cast_f64_to_f32(n2_, Ioovv.v, (float*)Ioovv.lp32, s);
  for (Ten* t : {&Iovov, &Ix})  // FP32 ring integrals transposed, read along k (staged in Tmp)
    if (t->lp32) {
      const int dims[4] = {o, v, o, v}, pm[4] = {2, 3, 0, 1};
      permute4(t->v, Tmp.v, dims, pm, 1.0, 0.0, s);
      cast_f64_to_f32(n2_, Tmp.v, (float*)t->lp32, s);
    }
  if (Ioovv.lp16) cast_f64_to_bf16(n2_, Ioovv.v, (uint16_t*)Ioovv.lp16, s);
  if (Iovov.lp16) {
    cast_f64_to_bf16_rows(ov, ov, ldov16_, Iovov.v, ov, (uint16_t*)Iovov.lp16, s);
    // Ix^T[(k,c)][(l,d)] = Ix[(l,d)][(k,c)] = (kd|lc), staged in Tmp
    const int dims[4] = {o, v, o, v};
    const int pm[4] = {0, 3, 2, 1};
    permute4(Iovov.v, Tmp.v, dims, pm, 1.0, 0.0, s);
    cast_f64_to_bf16_rows(ov, ov, ldov16_, Tmp.v, ov, (uint16_t*)Ix.lp16, s);
  }
  fill(ov_ + n2_, 0.0, zeros_, s);
  // f_ov == 0 lets A_F skip its singles-doubles coupling
  nrm_inf(ov, f_ov_, partials_ + reduce_partials_size(64) - 1, partials_, s);
  if (with_eigen) compute_eigen(foo, fvv, s);  // while the device works on the tensors above
  double fmax = 0.0;
  PNK_HIP(hipMemcpyAsync(&fmax, partials_ + reduce_partials_size(64) - 1, sizeof(double), hipMemcpyDeviceToHost, s));
  PNK_HIP(hipStreamSynchronize(s));
  fov_zero_ = (fmax == 0.0);
}

// --------------------------------------------------------- the program --

void Engine::run(Mode m) {
  mode_ = m;
  const int o = o_, v = v_, naux = naux_, np = np_;
  const int64_t O = o, V = v, ov = ov_, vv = V * V, oo = O * O;
  const int OV = (int)ov, OO = (int)oo, VV = (int)vv;

  const bool lowp = this->lowp();  // FP32 / BF16: the same sums, in the order the layouts below give
  const bool lowp_engine = opt_.lowp_f32 || opt_.lowp_bf16;

  // ---- T1 dressing: L~ = (1 - tau) L (1 + tau), slice naux is h ----
  mm(gd(np * o, o, v, v, 1, 1, v, o, 1, 1.0), Lov0, T1, Loo, &Loo0);                            // + L_kc t_i^c
  mm(batch0(gd(o, v, v, v, 1, 1, v, v, 1), np, 0, vv, ov), T1, Lvv0, Lvo, &Lvo0);               // + L_ab t_i^b
  mm(batch0(gd(v, o, o, 1, v, o, 1, 1, v, -1.0, 1.0), np, 0, oo, ov), T1, Loo, Lvo);            // - t_k^a L~_ki
  mm(batch0(gd(v, v, o, 1, v, v, 1, v, 1, -1.0), np, ov, 0, vv), Lov0, T1, Lvv, &Lvv0);         // - L_kc t_k^a

  // ---- dressed Fock F~ = h~ + sum_P [2 L~ D - L~_{:,o} L~_{o,:}] (F~_ai in R1) ----
  perm(Loo, LooT, 1, naux, o, o, 0, 2, 1, 3, 1.0, 0.0);
  dressed_fock_sums();
  mm(gd(o, o, naux * o, naux * O, 1, o, 1, o, 1, -1.0, 1.0), LooT, Loo, Foo);
  mm(gd(o, v, naux * o, naux * O, 1, v, 1, v, 1, -1.0, 1.0), LooT, Lov0, Fov);
  mm(gd(v, o, naux * o, 1, v, o, 1, 1, v, -1.0, 1.0), Lvo, Loo, R1);
  mm(gd(v, v, naux * o, 1, v, v, 1, v, 1, -1.0, 1.0), Lov0, Lvo, Fvv);                          // [c][a]

  // ---- amplitude layouts ----
  {
    AmpLayouts p{};
    p.t = out(T2);
    p.Tsia = out(Tsia); p.Uia = out(Uia);
    p.Tp = out(Tp); p.Tm = out(Tm); p.ldp = lad_.p2k; p.ldm = lad_.p2mk;
    p.diag = lowp ? 0.5 : 1.0;  // (FP64 has the half in S)
    // (an FP64 tangent has no use for the others)
    if (lowp_engine && (lowp || mode_ == Mode::Value)) {
      p.Tia = out(Tia); p.U = out(U); p.Uklca = out(Uklca); p.Uail = out(Uail);
    }
    amp_layouts(o, v, p, s_);
  }

  // ---- ladders, symmetry-adapted: for i <= j and the (anti)symmetric
  // combinations of c,d, R+ = T+ S, R- = T- A (the antisymmetric pairs over
  // i < j only: t_ii^cd = t_ii^dc) ----
  const int64_t P2 = lad_.p2, P2m = lad_.p2m, p2k = lad_.p2k, p2mk = lad_.p2mk, ldp = lad_.ldp, ldm = lad_.ldm;
  const int O2 = (int)lad_.o2, O2m = (int)lad_.o2m;
  const bool anti = P2m > 0 && O2m > 0;
  mm(gd(OO, OO, naux, 1, oo, oo, 1, oo, 1), Loo, Loo, Kilj);       // (ki|lj)~ as [(k,i)][(l,j)]
  if (lowp) {
    // S and A are symmetric matrices: read them along the contiguous index
    // the compute type stages best (n for FP32, k for BF16, whose copies'
    // rows are zero to their length, so that the packed amplitudes may run
    // the contraction over whole panels)
    const bool kc = jprec_ == Prec::BF16;
    const int64_t ls = kc ? ld16_ : ld32_, lm = kc ? ld16m_ : ld32m_;
    if (timers_) timers_->begin(kTimerPPL, s_);
    GemmDesc gs = gd(O2, (int)P2, (int)P2, p2k, 1, kc ? 1 : ls, kc ? ls : 1, ldp, 1);
    if (kc) gs.b_kzero = ld16_;
    mm(gs, Tp, S, Rp);
    if (anti) {
      GemmDesc ga = gd(O2m, (int)P2m, (int)P2m, p2mk, 1, kc ? 1 : lm, kc ? lm : 1, ldm, 1);
      if (kc) ga.b_kzero = ld16m_;
      mm(ga, Tm, Am, Rm);
    }
    if (timers_) timers_->end(kTimerPPL, s_);
    // hole-hole ladder
    mm(gd(OO, OO, VV, vv, 1, 1, vv, oo, 1), Ioovv, T2, Y);         // Y[(k,l)][(i,j)]
    perm(Kilj, Wkl, o, o, o, o, 0, 2, 1, 3, 1.0, 1.0, &Y);         // [(k,l)][(i,j)]
    mm(gd(OO, VV, OO, 1, oo, vv, 1, vv, 1), Wkl, T2, R2);
    // T1 part of the dressed ladder, Z[(i,j)][(k,b)]; BF16 reads the padded
    // copy of Wov
    GemmDesc gz = gd(OO, OV, VV, vv, 1, 1, kc ? ldw16_ : vv, ov, 1);
    if (kc) gz.b_kzero = ldw16_;
    mm(gz, T2, Wov, Z);
  } else {
    // further columns of S and A give Z and Y at half and a quarter of their
    // flops, and W_klij t_kl^ab acts on the pair combinations as well
    const double count = mm_flops_;
    if (timers_) timers_->begin(kTimerPPL, s_);
    mm(gd(O2, (int)ldp, (int)p2k, p2k, 1, ldp, 1, ldp, 1), Tp, S, Rp);
    if (anti) mm(gd(O2m, (int)ldm, (int)p2mk, p2mk, 1, ldm, 1, ldm, 1), Tm, Am, Rm);
    if (timers_) timers_->end(kTimerPPL, s_);
    LadderParts p{};
    p.l = lad_;
    p.Rp = out(Rp); p.Rm = out(Rm); p.Kilj = out(Kilj);
    p.Z = out(Z); p.Y = out(Y); p.Wp = out(Wp); p.Wm = out(Wm);
    p.Wkl = lowp_engine && mode_ == Mode::Value ? Wkl.v : nullptr;
    ladder_unpack(o, v, p, s_);
    // (columns past the pairs, whose Z and Y have been read, run along)
    mm(gd(O2, (int)p2k, (int)lad_.o2k, lad_.o2k, 1, p2k, 1, ldp, 1, 1.0, 1.0), Wp, Tp, Rp);
    if (anti) mm(gd(O2m, (int)p2mk, (int)lad_.o2mk, lad_.o2mk, 1, p2mk, 1, ldm, 1, 1.0, 1.0), Wm, Tm, Rm);
    // (counted in the form with whole Z, Y and W)
    mm_flops_ = count + 2.0 * O2 * P2 * P2 + 2.0 * O2m * P2m * P2m + 2.0 * oo * oo * vv + 2.0 * oo * vv * ov +
                2.0 * oo * oo * vv * (mode_ == Mode::Value ? 1.0 : 2.0);
  }

  // ---- Fock-type intermediates, Gv as [c][b] ----
  if (lowp) {
    mm(gd(v, v, (int)(oo * v), 1, v, 1, oo * V, v, 1, -1.0), Ikldc, Uail, Gv, &Fvv);
    mm(gd(o, o, (int)(O * vv), O * vv, 1, 1, O * vv, o, 1), Ioovv, U, Go, &Foo);
  } else {
    // u is symmetric in (k,b), (l,d): the sums over (l,d,k) and (c,l,d) run
    // along the rows of the ring's operands
    mm(gd(v, v, (int)(oo * v), 1, v, v, 1, v, 1, -1.0), Iovov, Uia, Gv, &Fvv);
    mm(gd(o, o, (int)(O * vv), O * vv, 1, 1, O * vv, o, 1), Iovov, Uia, Go, &Foo);
  }
  mm(gd((int)(oo * v), v, v, v, 1, v, 1, v, 1), T2, Gv, X);        // X = sum_c Gv_bc t_ij^ac
  mm(batch0(gd(o, VV, o, 1, o, vv, 1, vv, 1, -1.0, 1.0), o, 0, O * vv, O * vv), Go, T2, X);

  // ---- T1 part of the dressed ladder ----
  mm(batch0(gd(OO, v, o, 1, oo, v, 1, ov, 1, -0.5, 1.0), o, O * oo, 0, v), Y, T1, Z);
  mm(batch0(gd(v, v, o, 1, v, v, 1, v, 1, -1.0, 1.0), OO, 0, ov, vv), T1, Z, X);

  // ---- ring terms, rows and columns (i,a) ----
  // Engines that offer FP32 products keep J and K, the largest values these
  // round, as sums in ascending k from 1024 rows on: a last bit that depended
  // on the tiles moves single elements of an FP32 J v by an FP32 rounding (1e-8
  // of the largest, 1e-10 of the norm, at o = 16, v = 144 and 12/84; its error is
  // the same either way). It costs a residual 0.65 of 4.35 ms at 16/144, 2.0 of
  // 13.9 at 20/180 and 0.10 of 0.87 at 10/102. 1024 rows are 256 tiles in one
  // piece, one to a CU; below, where CUs would stay idle (44 of 318 us at 6/42),
  // the last bits follow the tiles.
  const bool f32_values = opt_.lowp_f32 && mode_ == Mode::Value && ov >= 1024;
  auto piece = [&](GemmDesc g) {
    g.ascending = f32_values;
    return g;
  };
  mm(piece(gd(OO, VV, naux, 1, oo, vv, 1, vv, 1)), Loo, Lvv, Tmp); // (ki|ac)~ as [(k,i)][(c,a)]
  perm(Tmp, K, o, o, v, v, 1, 3, 0, 2, 1.0, 0.0);                  // [(i,a)][(k,c)]
  const GemmDesc g0 = gd(OV, OV, naux, 1, ov, ov, 1, ov, 1), g1 = gd(OV, OV, OV, ov, 1, ov, 1, ov, 1),
                 gT = gd(OV, OV, OV, ov, 1, 1, ov, ov, 1);
  auto scaled = [](GemmDesc g, double alpha, double beta) {
    g.alpha = alpha;
    g.beta = beta;
    return g;
  };
  Ten KT = M;  // - K t in the tangent of M (J), free: a value pass has none yet, a tangent has read it by then
  KT.v = KT.d;
  const Ten* E = nullptr;
  double w = 0.0;
  if (lowp) {
    // (the copies of the ring integrals are read along k: transposed, but
    // for Iovov in BF16, which is symmetric)
    const bool kc16 = jprec_ == Prec::BF16;
    GemmDesc g = gd(OV, OV, OV, ov, 1, 1, kc16 ? ldov16_ : ov, ov, 1);
    if (kc16) g.b_kzero = ldov16_;
    mm(g0, Lvo, Lov0, J);                                          // (ai|kc)~
    mm(scaled(g, 0.5, 1.0), Uia, Iovov, J);
    mm(scaled(g, -0.5, 1.0), Tia, Ix, J);
    mm(scaled(g, -0.5, 1.0), Tsia, Ix, K);
    mm(gT, J, Uia, Tmp);                                           // J u_jk^bc
    mm(scaled(gT, -1.0, 1.0), K, Tia, Tmp);                        // - K t_kj^cb
    mm(scaled(gT, -1.0, 0.0), K, Tsia, KT);                        // - K_ki,bc t_kj^ac as [(i,b)][(j,a)]
    // (ai|bj)~: its (i,a),(j,b) and (j,b),(i,a) elements may differ by a
    // rounding, so it stays outside the pair sum, in the tangent of U, read
    // above only
    mm(g0, Lvo, Lvo, U);
    E = &U;
  } else {
    // With t = (u + s) / 2, s_jk^bc = t_jk^cb, and M = J - K / 2,
    //   J u - K t = M u - K s / 2,
    //   M = (ai|kc)~ - (ki|ac)~ / 2 + u ((kc|ld) - (kd|lc) / 2) / 2:
    // four products of ring size (six in a tangent) in place of six (nine)
    const int dims[4] = {o, v, o, v}, same[4] = {0, 1, 2, 3};
    if (f32_values) {
      mm(piece(g0), Lvo, Lov0, J);
      mm(piece(scaled(g1, 0.5, 1.0)), Uia, Iovov, J);
      mm(piece(scaled(g1, -0.5, 1.0)), Tia, Ix, J);
      mm(piece(scaled(g1, -0.5, 1.0)), Tsia, Ix, K);
      permute4(K.v, M.v, dims, same, -0.5, 1.0, s_, J.v);
      mm_flops_ -= 2.0 * ov * ov * ov;
    } else {
      mm(g0, Lvo, Lov0, M, &K, 0, -0.5);
      mm(scaled(g1, 0.5, 1.0), Uia, Lh, M);
      mm(scaled(g1, -0.5, 1.0), Tsia, Ix, K);
      if (lowp_engine && mode_ == Mode::Value) permute4(K.v, J.v, dims, same, 0.5, 1.0, s_, M.v);
    }
    mm(scaled(g0, 0.5, 0.0), Lvo, Lvo, Tmp);                       // (ai|bj)~ / 2, doubled by the pair sum
    mm(scaled(gT, 1.0, 1.0), M, Uia, Tmp);
    mm_flops_ += (mode_ == Mode::Value ? 2 : 3) * 2.0 * ov * ov * ov;  // (counted in the six-product form)
    mm(scaled(gT, -1.0, 0.0), K, Tsia, KT);
    w = 0.5;
  }

  // ---- r2 ----
  {
    DoublesParts p{};
    p.X = out(X); p.T = out(Tmp); p.S = out(KT); p.w = w; p.Rp = out(Rp); p.Rm = out(Rm); p.ldp = ldp; p.ldm = ldm;
    p.add = lowp;
    p.E = E ? out(*E) : nullptr;
    p.R = out(R2);
    doubles_sum(o, v, p, s_);
  }

  // ---- singles ----
  mm(gd(naux, OV, OV, ov, 1, ov, 1, ov, 1), Lov0, Uia, Q);         // Q[P][(i,c)]
  perm(Q, QT, 1, naux, o, v, 0, 2, 1, 3, 1.0, 0.0);
  mm(gd(o, v, naux * v, naux * V, 1, v, 1, v, 1, 1.0, 1.0), QT, Lvv, R1);
  mm(gd(OV, OO, naux, 1, ov, oo, 1, oo, 1), Lov0, Loo, Kilc);      // (ki|lc)~ as [(l,c)][(k,i)]
  if (lowp_engine && (lowp || mode_ == Mode::Value)) perm(Kilc, KilcT, o, v, o, o, 3, 2, 0, 1, 1.0, 0.0);
  if (lowp)  // sums over (k,l,c); over (l,c,k) in FP64, u symmetric as above
    mm(gd(o, v, (int)(oo * v), oo * V, 1, v, 1, v, 1, -1.0, 1.0), KilcT, Uklca, R1);
  else
    mm(gd(o, v, (int)(oo * v), 1, o, v, 1, v, 1, -1.0, 1.0), Kilc, Uia, R1);
  mm(gd(OV, 1, OV, ov, 1, 1, 1, 1, 1, 1.0, 1.0), Uia, Fov, R1);
}

// L~[naux] + 2 sum_P D_P L~[P] into Foo, Fov, R1 (F~_ai) and Fvv
void Engine::dressed_fock_sums() {
  const int naux = naux_, OV = (int)ov_;
  const Ten* L[4] = {&Loo, &Lov0, &Lvo, &Lvv};
  const Ten* F[4] = {&Foo, &Fov, &R1, &Fvv};
  const int n[4] = {o_ * o_, OV, OV, v_ * v_};
  if (lowp()) {
    trace_slices(naux, o_, Loo.d, D.d, s_);
    for (int q = 0; q < 4; ++q)
      mm(gd(1, n[q], naux, 0, 1, n[q], 1, 0, 1, 2.0), D, *L[q], *F[q], L[q], (int64_t)naux * n[q]);
    return;
  }
  FockSum p{};
  p.Loo = Loo.v;
  p.dLoo = mode_ == Mode::Tangent ? Loo.d : nullptr;
  for (int q = 0; q < 4; ++q) {
    p.n[q] = n[q];
    p.L[q] = L[q]->v;
    p.dL[q] = L[q]->d;
    p.F[q] = out(*F[q]);
    mm_flops_ += 2.0 * naux * n[q] * (p.dLoo && p.dL[q] ? 2.0 : 1.0);  // as one-row products
  }
  p.D = mode_ == Mode::Value ? D.v : nullptr;
  fock_sum(naux, o_, p, s_);
}

void Engine::residual(const double* t1, const double* t2, double* r1, double* r2, hipStream_t s) {
  s_ = s;
  T1.v = const_cast<double*>(t1);
  T2.v = const_cast<double*>(t2);
  R1.v = r1;
  R2.v = r2;
  if (timers_) timers_->begin(kTimerResidual, s);
  if (graph_ready(&res_slot_, t1, t2, r1, r2, Mode::Value)) PNK_HIP(hipGraphLaunch(res_slot_.exec, s));
  else run(Mode::Value);
  if (timers_) timers_->end(kTimerResidual, s);
}

void Engine::jvp(const double* x1, const double* x2, double* y1, double* y2, Prec prec, hipStream_t s) {
  PNK_REQUIRE(T1.v && T2.v, "jvp before any residual evaluation");
  PNK_REQUIRE(prec == Prec::F64 || (prec == Prec::F32 ? opt_.lowp_f32 : opt_.lowp_bf16),
              "internal: jvp in a precision the engine has no copies for");
  s_ = s;
  jprec_ = prec;
  if (timers_) timers_->begin(kTimerJvp, s);
  // graphs run on fixed tangent buffers: copy in, replay, copy out
  T1.d = tin_;
  T2.d = tin_ + ov_;
  R1.d = tout_;
  R2.d = tout_ + ov_;
  GraphSlot* slot = &jvp_slot_[(int)prec];
  if (graph_ready(slot, T1.v, T2.v, nullptr, nullptr, Mode::Tangent)) {
    jprec_ = prec;
    // (one copy each way when the caller's singles and doubles are adjacent)
    if (x2 == x1 + ov_) {
      PNK_HIP(hipMemcpyAsync(tin_, x1, (ov_ + n2_) * sizeof(double), hipMemcpyDeviceToDevice, s));
    } else {
      PNK_HIP(hipMemcpyAsync(tin_, x1, ov_ * sizeof(double), hipMemcpyDeviceToDevice, s));
      PNK_HIP(hipMemcpyAsync(tin_ + ov_, x2, n2_ * sizeof(double), hipMemcpyDeviceToDevice, s));
    }
    PNK_HIP(hipGraphLaunch(slot->exec, s));
    if (y2 == y1 + ov_) {
      PNK_HIP(hipMemcpyAsync(y1, tout_, (ov_ + n2_) * sizeof(double), hipMemcpyDeviceToDevice, s));
    } else {
      PNK_HIP(hipMemcpyAsync(y1, tout_, ov_ * sizeof(double), hipMemcpyDeviceToDevice, s));
      PNK_HIP(hipMemcpyAsync(y2, tout_ + ov_, n2_ * sizeof(double), hipMemcpyDeviceToDevice, s));
    }
  } else {
    T1.d = const_cast<double*>(x1);
    T2.d = const_cast<double*>(x2);
    R1.d = y1;
    R2.d = y2;
    run(Mode::Tangent);
  }
  if (timers_) timers_->end(kTimerJvp, s);
  mode_ = Mode::Value;
  jprec_ = Prec::F64;
}

void Engine::energy(const double* t1, const double* t2, double* e_dev, hipStream_t s) {
  pnk::energy(o_, v_, f_ov_, Itil.v, t1, t2, e_dev, partials_, s);
}

// (A_F x)_ij^ab = sum_c (f_ac x_ij^cb + f_bc x_ij^ac) - sum_k (f_ki x_kj^ab + f_kj x_ik^ab)
// (A_F x)_i^a   = sum_c f_ac x_i^c - sum_k f_ki x_k^a + sum_kc f_kc (2 x_ik^ac - x_ik^ca)
void Engine::fock_apply(const double* x1, const double* x2, double* y1, double* y2, hipStream_t s) {
  const int o = o_, v = v_;
  const int64_t O = o, V = v, vv = V * V, oo = O * O, ov = ov_;
  if (timers_) timers_->begin(kTimerFock, s);
  if (fop_ok_ && x1 != y1 && x2 != y2) {
    // virtual and occupied contractions and singles in one launch
    fock_op_apply(fop_, x1, x2, y1, y2, s);
  } else {
    // a index: batched over ij, y_ij = f_vv x_ij
    gemm64(with_ws(batch0(gd(v, v, v, v, 1, v, 1, v, 1), (int)oo, 0, vv, vv)), f_vv_, x2, y2, s);
    // b index: y[(ija)][b] += sum_c x[(ija)][c] f_bc
    gemm64(with_ws(gd((int)(oo * v), v, v, v, 1, 1, v, v, 1, 1.0, 1.0)), x2, f_vv_, y2, s);
    // i index: y[i][(jab)] -= sum_k f_ki x[k][(jab)]
    gemm64(with_ws(gd(o, (int)(O * vv), o, 1, o, O * vv, 1, O * vv, 1, -1.0, 1.0)), f_oo_, x2, y2, s);
    // j index: batched over i, y_i[j][(ab)] -= sum_k f_kj x_i[k][(ab)]
    gemm64(with_ws(batch0(gd(o, (int)vv, o, 1, o, vv, 1, vv, 1, -1.0, 1.0), o, 0, O * vv, O * vv)), f_oo_, x2, y2, s);
    // singles
    gemm64(with_ws(gd(o, v, v, v, 1, 1, v, v, 1)), x1, f_vv_, y1, s);
    gemm64(with_ws(gd(o, v, o, 1, o, v, 1, v, 1, -1.0, 1.0)), f_oo_, x1, y1, s);
  }
  if (!fov_zero_) {
    // u_x[i][a][k][c] = 2 x_ik^ac - x_ik^ca, then y1 += u_x f_ov
    const int dims[4] = {o, o, v, v};
    const int p1[4] = {0, 2, 1, 3};  // x_ik^ac at [i][a][k][c]
    const int p2[4] = {0, 3, 1, 2};  // x_ik^ca at [i][a][k][c]
    permute4(x2, Tmp.v, dims, p1, 2.0, 0.0, s);
    permute4(x2, Tmp.v, dims, p2, -1.0, 1.0, s);
    gemm64(with_ws(gd((int)ov, 1, (int)ov, ov, 1, 1, 1, 1, 1, 1.0, 1.0)), Tmp.v, f_ov_, y1, s);
  }
  if (timers_) timers_->end(kTimerFock, s);
}

}  // namespace pnk
