"""The inner solve A_F x = b in the eigenvectors of the Fock blocks: every form
of the rotation (either block diagonal already, the occupied position sets and
the full-layout form above 24 occupied orbitals), the packed and the full
layout, and solves longer than one and two segments of the recurrence."""

import numpy as np
import pytest
import torch

import paper_2608_06669_amd as pk
from gen import make_near_degenerate, make_problem, random_amplitudes
from gen.problems import haar_orthogonal
from oracle import solvers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def handle():
    h = pk.Handle(0)
    yield h
    h.close()


def dev(x):
    return torch.tensor(np.ascontiguousarray(x), device="cuda")


def host(x):
    return x.cpu().numpy()


@pytest.mark.parametrize("o,v", [(1, 9), (2, 20), (3, 8), (4, 17), (8, 36), (9, 41), (13, 24), (20, 17), (24, 12),
                                 (25, 11), (31, 8)])
@pytest.mark.parametrize("rotated", ["both", "occupied", "virtual", "none"])
@pytest.mark.parametrize("packed", [True, False])
def test_inner_solve_in_every_form(handle, o, v, rotated, packed):
    """rtol 1e-12 and a condition number below 6 leave 1e-11 of the largest
    component; the margin to 1e-10 is for the rotations' rounding."""
    p = make_problem(o, v, 12, 900 + o, gauge="haar")
    if rotated in ("virtual", "none"):
        p.f_oo[:] = np.diag(np.linalg.eigvalsh(p.f_oo))
    if rotated in ("occupied", "none"):
        p.f_vv[:] = np.diag(np.linalg.eigvalsh(p.f_vv))
    P = pk.DeviceProblem.from_problem(p)
    for seed in (1, 2):
        b1, b2 = random_amplitudes(o, v, seed, scale=1.0)
        if not packed:
            b2 = np.random.default_rng(seed).standard_normal(b2.shape)  # no pair symmetry
        x1, x2, iters, ok = handle.precond_solve(P, dev(b1), dev(b2), rtol=1e-12, maxit=300, pair_symmetric=packed)
        e1, e2 = solvers.fock_solve_exact(p.f_oo, p.f_ov, p.f_vv, b1, b2)
        assert ok and 0 < iters <= 300
        assert np.abs(host(x1) - e1).max() <= 1e-10 * np.abs(e1).max()
        assert np.abs(host(x2) - e2).max() <= 1e-10 * np.abs(e2).max()


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("lowest,at_least", [(1e-2, 65), (1e-3, 129)])
def test_inner_solve_over_several_segments(handle, packed, lowest, at_least):
    """Orbital energies that fall geometrically towards the gap take more steps
    than one (64) and two segments hold; the residual, formed with the A_F
    product, meets the tolerance."""
    p = make_near_degenerate(4, 30, 12, 77)
    rng = np.random.default_rng(6)
    uo, uv = haar_orthogonal(rng, 4), haar_orthogonal(rng, 30)
    p.f_oo[:] = -(uo * np.geomspace(lowest, 1.5, 4)) @ uo.T
    p.f_vv[:] = (uv * np.geomspace(lowest, 2.5, 30)) @ uv.T
    p.f_oo[:] = 0.5 * (p.f_oo + p.f_oo.T)
    p.f_vv[:] = 0.5 * (p.f_vv + p.f_vv.T)
    P = pk.DeviceProblem.from_problem(p)
    b1, b2 = random_amplitudes(4, 30, 5, scale=1.0)
    d1, d2 = dev(b1), dev(b2)
    for _ in range(2):  # the second replays the recorded launches
        x1, x2, iters, ok = handle.precond_solve(P, d1, d2, rtol=1e-11, maxit=2000, pair_symmetric=packed)
        assert ok and iters >= at_least
        y1, y2 = handle.fock_apply(P, x1, x2)
        r = torch.sqrt(((d1 - y1) ** 2).sum() + ((d2 - y2) ** 2).sum())
        b = torch.sqrt((d1 ** 2).sum() + (d2 ** 2).sum())
        # (the product itself rounds at 1e-15 of ||A_F|| ||x||, 1e-12 here)
        assert float(r / b) <= 2e-11


def test_inner_solve_stops_at_its_cap(handle):
    p = make_near_degenerate(4, 30, 12, 77, gap=0.004)
    P = pk.DeviceProblem.from_problem(p)
    b1, b2 = random_amplitudes(4, 30, 5, scale=1.0)
    for maxit in (1, 63, 64, 65, 100):
        x1, x2, iters, ok = handle.precond_solve(P, dev(b1), dev(b2), rtol=1e-13, maxit=maxit, pair_symmetric=True)
        # (whole blocks of four launches, the first of which completes no step)
        assert not ok and iters == 4 * -(-maxit // 4) - 1
        assert np.isfinite(host(x2)).all()


@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("o,v,lowest,at_least", [(2, 5, 1e-3, 20), (4, 20, 1e-2, 65), (3, 36, 1e-3, 129), (4, 28, 1e-3, 129)])
def test_inner_solve_in_one_workgroup(handle, o, v, lowest, at_least, packed):
    """Vectors short enough for one workgroup, over one and several segments,
    and a step limit that ends the solve before the tolerance."""
    p = make_near_degenerate(o, v, 12, 78)
    rng = np.random.default_rng(7)
    uo, uv = haar_orthogonal(rng, o), haar_orthogonal(rng, v)
    p.f_oo[:] = -(uo * np.geomspace(lowest, 1.5, o)) @ uo.T
    p.f_vv[:] = (uv * np.geomspace(lowest, 2.5, v)) @ uv.T
    p.f_oo[:] = 0.5 * (p.f_oo + p.f_oo.T)
    p.f_vv[:] = 0.5 * (p.f_vv + p.f_vv.T)
    P = pk.DeviceProblem.from_problem(p)
    b1, b2 = (dev(b) for b in random_amplitudes(o, v, 6, scale=1.0))
    x1, x2, iters, ok = handle.precond_solve(P, b1, b2, rtol=1e-11, maxit=2000, pair_symmetric=packed)
    assert ok and iters >= at_least
    y1, y2 = handle.fock_apply(P, x1, x2)
    r = torch.sqrt(((b1 - y1) ** 2).sum() + ((b2 - y2) ** 2).sum())
    # (the product itself rounds at 1e-15 of ||A_F|| ||x||, 1e-12 here)
    assert float(r / torch.sqrt((b1 ** 2).sum() + (b2 ** 2).sum())) <= 2e-11
    _, _, short, ok = handle.precond_solve(P, b1, b2, rtol=1e-11, maxit=6, pair_symmetric=packed)
    assert not ok and 6 <= short <= 8
