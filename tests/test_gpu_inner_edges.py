"""The inner solve on right-hand sides and Fock blocks that are not finite: it
ends, says that it has not converged, and leaves the handle as it was. Both
forms of the recurrence (one workgroup, a launch for each step), both layouts.
And FP32 and BF16 tangents with one occupied orbital, whose buffers have a
rule of their own."""

import numpy as np
import pytest
import torch

import paper_2608_06669_amd as pk
from gen import make_problem, random_amplitudes
from oracle import ccsd, solvers

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.tensor(np.ascontiguousarray(x), device="cuda")


@pytest.fixture(scope="module")
def handle():
    h = pk.Handle(0)
    yield h
    h.close()


@pytest.mark.parametrize("o,v", [(2, 9), (8, 36)])
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("where", ["b1", "b2", "f_oo", "f_vv"])
def test_not_finite(handle, o, v, packed, bad, where):
    """The solve after it, of finite arrays, as exact as ever (rtol 1e-12 and a
    condition number below 6 leave 1e-11; the margin to 1e-10 is for the
    rotations)."""
    p = make_problem(o, v, 12, 90 + o, gauge="haar")
    P = pk.DeviceProblem.from_problem(p)
    b1, b2 = random_amplitudes(o, v, 3, scale=1.0)
    c1, c2, q = b1.copy(), b2.copy(), make_problem(o, v, 12, 90 + o, gauge="haar")
    {"b1": c1, "b2": c2, "f_oo": q.f_oo, "f_vv": q.f_vv}[where].flat[0] = bad
    _, _, iters, ok = handle.precond_solve(pk.DeviceProblem.from_problem(q), dev(c1), dev(c2), rtol=1e-12, maxit=40,
                                           pair_symmetric=packed)
    assert not ok and 0 <= iters <= 48
    x1, x2, _, ok = handle.precond_solve(P, dev(b1), dev(b2), rtol=1e-12, maxit=300, pair_symmetric=packed)
    e1, e2 = solvers.fock_solve_exact(p.f_oo, p.f_ov, p.f_vv, b1, b2)
    assert ok
    assert np.abs(x1.cpu().numpy() - e1).max() <= 1e-10 * np.abs(e1).max()
    assert np.abs(x2.cpu().numpy() - e2).max() <= 1e-10 * np.abs(e2).max()


@pytest.mark.parametrize("prec,rel", [("fp32", 5e-5), ("bf16", 3e-2)])
@pytest.mark.parametrize("v,naux", [(1, 2), (2, 5), (32, 3), (65, 70)])
def test_low_precision_tangent_with_one_occupied_orbital(handle, v, naux, prec, rel):
    """Unit roundoff (2^-24, 2^-8) over contractions of a few thousand terms;
    the FP64 residual and J v of the same engine within 1e-10."""
    p = make_problem(1, v, naux, 63 + v, gauge="haar")
    t1, t2 = random_amplitudes(1, v, 64, scale=0.02)
    v1, v2 = random_amplitudes(1, v, 65, scale=1.0)
    P, args = pk.DeviceProblem.from_problem(p), (p.f_oo, p.f_ov, p.f_vv, p.L, t1, t2)
    want = ccsd.jvp_complex_step(*args, v1, v2)
    for pr, bound in ((prec, rel), ("fp64", 1e-10), (prec, rel)):
        got = handle.jvp(P, dev(t1), dev(t2), dev(v1), dev(v2), prec=pr)
        num = sum(np.sum((g.cpu().numpy() - w) ** 2) for g, w in zip(got, want))
        assert np.sqrt(num / sum(np.sum(w ** 2) for w in want)) < bound
