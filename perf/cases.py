"""The work that the solver's speed is measured on: single evaluations of the
coupled-cluster residual, its Jacobian products and the preconditioner, whole
Newton-Krylov solves and a batch of serving requests, each through the
package's public entry points.

Sizes are those of the shipped configurations (o/v/naux = 4/16/48, 10/90/300,
16/144/480, 20/180/600) and of the serving stream (o 4..16, v 5..9 times o,
naux = 3 (o + v), jittered to odd values in the drawn cases). Single
evaluations take the configurations' integrals (sigma 0.05). Whole solves take
integrals scaled to the correlation energy of a molecule (`weak_sigma`), so
that every seed converges, as a user's solves do.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2608_06669_amd as pk


def _case(name, kind, o, v, naux, **kw):
    return dict(name=name, kind=kind, o=o, v=v, naux=naux, **kw)


def listed():
    return [
        # one residual of a minimal-basis molecule: launches and latency
        _case("residual_4_16", "residual", 4, 16, 48, gauge="canonical"),
        # a residual of a serving-stream request with odd sizes
        _case("residual_13_91", "residual", 13, 91, 311, gauge="haar"),
        # the residual at the largest shipped configuration
        _case("residual_20_180", "residual", 20, 180, 600, gauge="haar"),
        # Jacobian products, one per precision the solver offers
        _case("jvp_f64_10_90", "jvp", 10, 90, 300, gauge="haar", prec="fp64"),
        _case("jvp_f32_16_144", "jvp", 16, 144, 480, gauge="haar", prec="fp32"),
        _case("jvp_bf16_20_180", "jvp", 20, 180, 600, gauge="haar", prec="bf16"),
        # the preconditioner's inverse inside a Newton step: the tolerance of
        # the right-hand side, on pair-symmetric vectors
        _case("precond_10_90", "precond", 10, 90, 300, gauge="haar", rtol=1e-12),
        _case("precond_20_180", "precond", 20, 180, 600, gauge="haar", rtol=1e-12),
        # a whole solve of a minimal-basis molecule: host steps and launches
        _case("solve_4_16", "solve", 4, 16, 48, gauge="canonical", prec="fp64", inner_rtol_jv=0.0),
        # a whole solve in a localised (rotated) gauge, all in 64 bits
        _case("solve_10_90", "solve", 10, 90, 300, gauge="haar", prec="fp64", inner_rtol_jv=0.0),
        # the headline: a whole solve with BF16 Jacobian products
        _case("solve_bf16_20_180", "solve", 20, 180, 600, gauge="haar", prec="bf16", inner_rtol_jv=1e-4),
        # six requests of the serving stream, four at once
        _case("serve_6", "serve", 9, 63, 216, gauge="haar", prec="bf16", inner_rtol_jv=1e-4, requests=6),
    ]


def draw(rng):
    kind = rng.choice(["residual", "residual", "jvp", "jvp", "jvp", "precond", "precond", "solve", "solve", "serve"])
    top = {"solve": 14, "serve": 10}.get(kind, 20)
    o = int(round(math.exp(rng.uniform(math.log(3), math.log(top)))))
    v = int(round(o * rng.uniform(4.0, 9.0))) + rng.choice([0, 0, 1])
    naux = 3 * (o + v) + rng.choice([0, 0, -1, 1, 5])
    c = dict(kind=kind, o=o, v=v, naux=naux, gauge=rng.choice(["canonical", "haar"]))
    if kind in ("jvp", "solve", "serve"):
        c["prec"] = rng.choice(["fp64", "fp32", "bf16"])
    if kind == "precond":
        c["rtol"] = rng.choice([1e-4, 1e-8, 1e-12])
    if kind in ("solve", "serve"):
        c["inner_rtol_jv"] = {"fp64": 0.0, "fp32": 1e-6, "bf16": 1e-4}[c["prec"]]
    if kind == "serve":
        c["requests"] = rng.randint(2, 6)
    return c


# ------------------------------------------------------------- inputs ----

def weak_sigma(o, v, naux):
    """Spread of the factors L at which the correlation energy is about 0.15
    Hartree for each occupied orbital: the second-order energy grows as
    o^2 v^2 naux sigma^4."""
    return (0.4 * o / (float(o * v) ** 2 * naux)) ** 0.25


def _haar(rng, m):
    q, r = np.linalg.qr(rng.standard_normal((m, m)))
    return q * np.sign(np.diag(r))[None, :]


def _arrays(o, v, naux, gauge, sigma, seed):
    """f_oo, f_ov, f_vv, L on the GPU: orbital energies in [-1.5, -0.5] and
    [0.3, 2.5], symmetric Gaussian factors."""
    rng = np.random.default_rng(seed)
    f_oo = np.diag(np.sort(rng.uniform(-1.5, -0.5, o)))
    f_vv = np.diag(np.sort(rng.uniform(0.3, 2.5, v)))
    if gauge == "haar":
        uo, uv = _haar(rng, o), _haar(rng, v)
        f_oo, f_vv = uo @ f_oo @ uo.T, uv @ f_vv @ uv.T
        f_oo, f_vv = 0.5 * (f_oo + f_oo.T), 0.5 * (f_vv + f_vv.T)
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(naux, o + v, o + v, dtype=torch.float64, device="cuda", generator=g) * sigma
    L = torch.triu(x) + torch.triu(x, 1).transpose(1, 2)
    return (torch.tensor(f_oo, device="cuda"), torch.zeros(o, v, dtype=torch.float64, device="cuda"),
            torch.tensor(f_vv, device="cuda"), L.contiguous())


def _vector(o, v, seed, scale):
    """A pair-symmetric amplitude-like vector."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x1 = scale * torch.randn(o, v, dtype=torch.float64, device="cuda", generator=g)
    x2 = scale * torch.randn(o, o, v, v, dtype=torch.float64, device="cuda", generator=g)
    return x1, (0.5 * (x2 + x2.permute(1, 0, 3, 2))).contiguous()


def _host(arrays):
    a, b, c, d = (x.cpu().numpy() for x in arrays)
    return SimpleNamespace(f_oo=a, f_ov=b, f_vv=c, L=d)


def _request_shapes(case):
    """The requests' sizes around the case's: o falls from one to the next."""
    return [(max(2, case["o"] - k), max(4, case["v"] - 5 * k), max(8, case["naux"] - 13 * k))
            for k in range(case["requests"])]


def _inputs(case, seed):
    o, v, naux, kind = case["o"], case["v"], case["naux"], case["kind"]
    if kind == "serve":
        return [_arrays(a, b, n, case["gauge"], weak_sigma(a, b, n), 1000 * seed + k)
                for k, (a, b, n) in enumerate(_request_shapes(case))]
    sigma = 0.05 if kind != "solve" else weak_sigma(o, v, naux)
    arrays = _arrays(o, v, naux, case["gauge"], sigma, seed)
    if kind == "residual":
        return arrays, _vector(o, v, 2 * seed + 1, 0.05)
    if kind == "jvp":
        return arrays, _vector(o, v, 2 * seed + 1, 0.05), _vector(o, v, 3 * seed + 2, 1.0)
    if kind == "precond":
        return arrays, _vector(o, v, 2 * seed + 1, 1.0)
    return (arrays,)


def _options(case):
    return dict(tol_inf=1e-10, jvp_prec=case["prec"], inner_rtol_jv=case["inner_rtol_jv"])


def prepare(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "serve":
        return dict(case=case, server=pk.Server(0, mem_budget=16 << 30, max_slots=4), problems=[_host(p) for p in x])
    return dict(case=case, handle=pk.Handle(0), problem=pk.DeviceProblem.from_problem(_host(x[0])), vectors=x[1:])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        srv = state["server"]
        ids = [srv.submit(p, **_options(case)) for p in state["problems"]]
        srv.drain()
        got = [srv.poll(i) for i in ids]
        return [(g["e_corr"], g["t1"], g["t2"]) for g in got]
    h, p, vec = state["handle"], state["problem"], state["vectors"]
    if kind == "residual":
        (t1, t2), = vec
        return h.residual(p, t1, t2)
    if kind == "jvp":
        (t1, t2), (v1, v2) = vec
        return h.jvp(p, t1, t2, v1, v2, prec=case["prec"])
    if kind == "precond":
        (b1, b2), = vec
        x1, x2, _, _ = h.precond_solve(p, b1, b2, rtol=case["rtol"], maxit=200, pair_symmetric=True)
        return x1, x2
    t1, t2, info = h.solve_pnk(p, **_options(case))
    return info["e_corr"], t1, t2


# --------------------------------------------------------------- work ----

def _residual_flops(o, v, naux):
    """Products of one residual: the ladder over (anti)symmetric pairs, six
    ring-sized products, the hole-hole ladder, the factors' products."""
    p2, m2, oo = v * (v + 1) // 2, v * (v - 1) // 2, o * (o + 1) // 2
    return (2.0 * oo * p2 * p2 + 2.0 * (o * (o - 1) // 2) * m2 * m2 + 12.0 * (o * v) ** 3 + 4.0 * o ** 4 * v ** 2
            + 2.0 * o ** 3 * v ** 3 + 8.0 * naux * (o * v) ** 2 + 4.0 * (o * v) ** 2 * (o + v)
            + 4.0 * naux * o * v * (o + v))


def _precond_flops(o, v):
    """One product with the Fock operator on pairs i <= j."""
    return 2.0 * o * (o + 1) * v * v * (o + v)


def work(case):
    o, v, naux, kind = case["o"], case["v"], case["naux"], case["kind"]
    vec = 8.0 * (o * v + (o * v) ** 2)
    ints = 8.0 * (naux * (o + v) ** 2 + o * o + v * v + o * v)
    if kind == "residual":
        return dict(bytes=ints + 2 * vec, flops=_residual_flops(o, v, naux))
    if kind == "jvp":
        return dict(bytes=ints + 3 * vec, flops=2.5 * _residual_flops(o, v, naux))
    if kind == "precond":
        # about one Krylov step for each half digit, on half the pairs
        steps = max(1.0, -2.0 * math.log10(case["rtol"]))
        return dict(bytes=ints + 2 * vec + steps * 2 * vec, flops=steps * _precond_flops(o, v))
    # a solve: about six Newton steps of four Jacobian products each
    shapes = _request_shapes(case) if kind == "serve" else [(o, v, naux)]
    total = dict(bytes=0.0, flops=0.0)
    for a, b, n in shapes:
        one = 8.0 * (a * b + (a * b) ** 2)
        total["bytes"] += 8.0 * n * (a + b) ** 2 + 60 * one
        total["flops"] += 42 * _residual_flops(a, b, n) + 300 * _precond_flops(a, b)
    return total


# -------------------------------------------------- 64-bit references ----

def _es(spec, *ops):
    return torch.einsum(spec, *ops)


def _mean_field(L, o):
    """sum_k 2 (pq|kk) - (pk|kq)"""
    naux, n = L.shape[0], L.shape[1]
    d = L[:, :o, :o].diagonal(dim1=1, dim2=2).sum(1)
    left = L[:, :, :o].permute(1, 0, 2).reshape(n, naux * o)
    right = L[:, :o, :].reshape(naux * o, n)
    return 2.0 * (d @ L.reshape(naux, n * n)).reshape(n, n) - left @ right


def _residual64(f, L, o, t1, t2):
    """Singles and doubles of exp(-T) H exp(T)|0> for a closed shell, from
    factors dressed with the singles: X -> (1 - t) X (1 + t)."""
    v, n, naux = t1.shape[1], f.shape[0], L.shape[0]
    ov = o * v
    tau = torch.zeros(n, n, dtype=f.dtype, device=f.device)
    tau = torch.cat([tau[:o], torch.cat([t1.T, tau[o:, o:]], 1)], 0)
    eye = torch.eye(n, dtype=f.dtype, device=f.device)
    h = (eye - tau) @ (f - _mean_field(L, o)) @ (eye + tau)
    Lt = torch.matmul(torch.matmul(eye - tau, L), eye + tau)
    F = h + _mean_field(Lt, o)
    Foo, Fov, Fvo, Fvv = F[:o, :o], F[:o, o:], F[o:, :o], F[o:, o:]
    Loo, Lov = Lt[:, :o, :o].reshape(naux, o * o), Lt[:, :o, o:].reshape(naux, ov)
    Lvo, Lvv = Lt[:, o:, :o].reshape(naux, ov), Lt[:, o:, o:].reshape(naux, v * v)
    u = 2.0 * t2 - t2.transpose(2, 3)
    kcld = (Lov.T @ Lov).reshape(o, v, o, v)
    klcd = kcld.permute(0, 2, 1, 3).reshape(o * o, v * v)
    # singles
    q = (Lov @ u.permute(1, 3, 0, 2).reshape(ov, ov)).reshape(naux, o, v)  # [P][i][c]
    kilc = (Loo.T @ Lov).reshape(o, o, o, v)
    r1 = (Fvo.T + q.permute(1, 0, 2).reshape(o, naux * v)
          @ Lvv.reshape(naux, v, v).permute(0, 2, 1).reshape(naux * v, v)
          - kilc.permute(1, 0, 2, 3).reshape(o, o * o * v) @ u.permute(0, 1, 3, 2).reshape(o * o * v, v)
          + (u.permute(0, 2, 1, 3).reshape(ov, ov) @ Fov.reshape(ov)).reshape(o, v))
    # doubles
    t_ij = t2.reshape(o * o, v * v)
    W = ((Loo.T @ Loo).reshape(o, o, o, o).permute(0, 2, 1, 3).reshape(o * o, o * o) + klcd @ t_ij.T)
    ladder = []
    for a0 in range(0, v, 16):
        la = Lvv.reshape(naux, v, v)[:, a0:a0 + 16, :]
        na = la.shape[1]
        w = (la.reshape(naux, na * v).T @ Lvv).reshape(na, v, v, v)  # [a][c][b][d]
        ladder.append((t_ij @ w.permute(1, 3, 0, 2).reshape(v * v, na * v)).reshape(o * o, na, v))
    r2 = ((Lvo.T @ Lvo).reshape(v, o, v, o).permute(1, 3, 0, 2) + torch.cat(ladder, 1).reshape(o, o, v, v)
          + (W.T @ t_ij).reshape(o, o, v, v))
    Gv = Fvv - _es("klcd,klbd->bc", klcd.reshape(o, o, v, v), u)
    Go = Foo + _es("klcd,jlcd->kj", klcd.reshape(o, o, v, v), u)
    u_ld = u.permute(0, 2, 1, 3).reshape(ov, ov)          # u_il^ad as [(i,a)][(l,d)]
    t_ld = t2.permute(0, 2, 1, 3).reshape(ov, ov)
    s_ld = t2.permute(0, 3, 1, 2).reshape(ov, ov)         # t_il^da as [(i,a)][(l,d)]
    I = kcld.reshape(ov, ov)
    X = kcld.permute(2, 1, 0, 3).reshape(ov, ov)          # (kd|lc) as [(l,d)][(k,c)]
    J = (Lvo.reshape(naux, v, o).permute(0, 2, 1).reshape(naux, ov).T @ Lov + 0.5 * u_ld @ I - 0.5 * t_ld @ X)
    K = ((Loo.T @ Lvv).reshape(o, o, v, v).permute(1, 2, 0, 3).reshape(ov, ov) - 0.5 * s_ld @ X)  # [(i,a)][(k,c)]
    x = (t2.reshape(o * ov, v) @ Gv.T).reshape(o, o, v, v)
    x = x - _es("kj,ikab->ijab", Go, t2)
    kc_jb = u.permute(1, 3, 0, 2).reshape(ov, ov)         # u_jk^bc as [(k,c)][(j,b)]
    x = x + (J @ kc_jb).reshape(o, v, o, v).permute(0, 2, 1, 3)
    x = x - (K @ t_ld).reshape(o, v, o, v).permute(0, 2, 1, 3)
    x = x - (K @ s_ld).reshape(o, v, o, v).permute(0, 2, 3, 1)
    return r1, r2 + x + x.permute(1, 0, 3, 2)


def _energy64(f_ov, L, t1, t2):
    o, v = t1.shape
    lov = L[:, :o, o:].reshape(L.shape[0], o * v)
    g = (lov.T @ lov).reshape(o, v, o, v).permute(0, 2, 1, 3)
    tau = t2 + t1[:, None, :, None] * t1[None, :, None, :]
    return 2.0 * (f_ov * t1).sum() + (g * (2.0 * tau - tau.transpose(2, 3))).sum()


def _fock64(f_oo, f_ov, f_vv):
    return torch.cat([torch.cat([f_oo, f_ov], 1), torch.cat([f_ov.T, f_vv], 1)], 0)


def _rotate(uo, uv, x1, x2):
    """x with every index contracted with a row index of uo, uv."""
    o, v = x1.shape
    y = (uo.T @ x2.reshape(o, -1)).reshape(o, o, v, v)
    y = torch.matmul(uo.T, y.reshape(o, o, v * v)).reshape(o, o, v, v)
    return uo.T @ x1 @ uv, torch.matmul(torch.matmul(uv.T, y), uv)


def _denominators(eo, ev):
    d1 = ev[None, :] - eo[:, None]
    return d1, d1[:, None, :, None] + d1[None, :, None, :]


def _levels(f):
    """Eigenvalues and eigenvectors of a small symmetric matrix."""
    e, u = np.linalg.eigh(f.cpu().numpy())
    return torch.tensor(e, device=f.device), torch.tensor(u, device=f.device)


def _solve64(f_oo, f_ov, f_vv, L):
    """The amplitudes at which the residual vanishes, by extrapolated
    fixed-point steps in the orbitals that make f diagonal."""
    (eo, uo), (ev, uv) = _levels(f_oo), _levels(f_vv)
    o = eo.shape[0]
    u = torch.block_diag(uo, uv)
    f, Lc = torch.diag(torch.cat([eo, ev])), u.T @ L @ u
    Lc = 0.5 * (Lc + Lc.transpose(1, 2))
    d1, d2 = _denominators(eo, ev)
    t1, t2 = torch.zeros_like(d1), torch.zeros_like(d2)
    past, last = [], math.inf
    for _ in range(100):
        r1, r2 = _residual64(f, Lc, o, t1, t2)
        size = float(torch.sqrt(r1.square().sum() + r2.square().sum()))
        if size < 1e-14 * math.sqrt(r2.numel()) or (size < 1e-10 and size > 0.9 * last):
            break
        last = size
        e1, e2 = -r1 / d1, -r2 / d2
        past = (past + [(t1 + e1, t2 + e2, e1, e2)])[-8:]
        m = len(past)
        g = np.zeros((m + 1, m + 1))
        g[m, :m] = g[:m, m] = 1.0
        for a in range(m):
            for b in range(m):
                g[a, b] = float((past[a][2] * past[b][2]).sum() + (past[a][3] * past[b][3]).sum())
        scale = max(np.abs(np.diag(g)[:m]).max(), 1e-300)
        g[:m, :m] /= scale
        c = np.linalg.lstsq(g, np.eye(m + 1)[m], rcond=None)[0][:m]
        t1 = sum(w * p[0] for w, p in zip(c, past))
        t2 = sum(w * p[1] for w, p in zip(c, past))
    e = _energy64(torch.zeros_like(d1), Lc, t1, t2)
    t1, t2 = _rotate(uo.T, uv.T, t1, t2)
    return float(e), t1, t2.contiguous()


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "serve":
        return [tuple(r if isinstance(r, float) else r.cpu().numpy() for r in _solve64(*p)) for p in x]
    f_oo, f_ov, f_vv, L = x[0]
    if kind == "solve":
        return _solve64(f_oo, f_ov, f_vv, L)
    if kind == "precond":
        (eo, uo), (ev, uv) = _levels(f_oo), _levels(f_vv)
        d1, d2 = _denominators(eo, ev)
        b1, b2 = _rotate(uo, uv, *x[1])
        y1, y2 = _rotate(uo.T, uv.T, b1 / d1, b2 / d2)
        return y1, y2.contiguous()
    f, o = _fock64(f_oo, f_ov, f_vv), case["o"]
    if kind == "residual":
        r1, r2 = _residual64(f, L, o, *x[1])
        return r1, r2.contiguous()
    _, (j1, j2) = torch.func.jvp(lambda a, b: _residual64(f, L, o, a, b), x[1], x[2])
    return j1, j2.contiguous()
