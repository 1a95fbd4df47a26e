"""The FP64 product's other forms, A B + A2 B2 in one sum, C from another
array than Cin, and sums in ascending k, at the edges of its panels and chunks,
against numpy's float64 products (the bound is that of any order of summation:
a relative 2^-53 for each of the terms that a sum holds)."""

import numpy as np
import pytest
import torch

import paper_2608_06669_amd as pk

pytestmark = pytest.mark.gpu

# (M, N, K, nbatch, splitk): the short-contraction kernel; remainder panels
# alone (K < 8); whole panels alone; remainders of 1 and 7 columns over 1 to 9
# panels; chunks, a cut tail after whole rounds, tiles of 48, 72 and 80 rows
SIZES = [(5, 90, 20, 2, False), (70, 66, 5, 2, False), (40, 65, 8, 1, False), (65, 130, 17, 3, False),
         (66, 64, 72, 1, False), (130, 62, 39, 2, False), (20, 18, 4001, 1, True), (1100, 1090, 96, 1, True),
         (48, 130, 40, 1, False), (143, 66, 100, 1, True), (79, 129, 1001, 1, True)]


def _operand(x, kc, odd):
    """The batch x [nb][rows][K], NaN between its rows and before it. Returns
    (tensor view, strides of rows, k and batch)."""
    nb, rows, K = x.shape
    y = x if kc else x.transpose(0, 2, 1)
    ld = y.shape[2] + 2 + (y.shape[2] % 2 != odd)
    buf = np.full((nb, y.shape[1], ld), np.nan)
    buf[:, :, : y.shape[2]] = y
    t = torch.tensor(np.concatenate([np.full(odd, np.nan), buf.ravel()]), device="cuda")[odd:]
    return t, (ld if kc else 1), (1 if kc else ld), y.shape[1] * ld


@pytest.mark.parametrize("M,N,K,nb,splitk", SIZES)
@pytest.mark.parametrize("akc,bkc", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("odd", [0, 1])
def test_two_products_and_another_input(M, N, K, nb, splitk, akc, bkc, odd):
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, A2 = rng.standard_normal((2, nb, M, K))
    B, B2 = rng.standard_normal((2, nb, N, K))
    Cin = rng.standard_normal((nb, M, N))
    ta, *sa = _operand(A, akc, odd)
    tb, *sb = _operand(B, bkc, odd)
    ta2, tb2 = _operand(A2, akc, odd)[0], _operand(B2, bkc, odd)[0]
    cin = torch.tensor(Cin, device="cuda")
    for two in (True, False):
        out = torch.full_like(cin, float("nan"))
        pk.api.diag_gemm_forms(ta, tb, out, sa, (sb[1], sb[0], sb[2]), (N, 1, M * N), M, N, K, nb,
                               A2=ta2 if two else None, B2=tb2 if two else None, Cin=cin, alpha=-0.5, beta=2.0,
                               splitk=splitk)
        f = 1.0 if two else 0.0
        ref = -0.5 * (A @ B.transpose(0, 2, 1) + f * A2 @ B2.transpose(0, 2, 1)) + 2.0 * Cin
        size = 0.5 * (np.abs(A) @ np.abs(B.transpose(0, 2, 1)) + f * np.abs(A2) @ np.abs(B2.transpose(0, 2, 1)))
        size += 2.0 * np.abs(Cin)
        err = np.abs(out.cpu().numpy() - ref)
        assert (err <= 2 * (2 * K + 4) * 2.0 ** -53 * size).all(), (two, float((err / size).max()))
    assert np.array_equal(cin.cpu().numpy(), Cin)


@pytest.mark.parametrize("K", [5, 8, 39, 1001])
@pytest.mark.parametrize("akc", [True, False])
@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("two", [True, False])
def test_ascending_sums_do_not_depend_on_the_tiles(K, akc, odd, two):
    """79 rows (tiles of 80 where the order is free) and 20 (cut along k where
    it is), the rows of the larger product bit for bit."""
    rng = np.random.default_rng(K)
    A, A2 = rng.standard_normal((2, 1, 79, K))
    B, B2 = rng.standard_normal((2, 1, 150, K))
    got = []
    for rows in (79, 20):
        ta, *sa = _operand(A[:, :rows], akc, odd)
        tb, *sb = _operand(B, False, odd)
        ta2, tb2 = _operand(A2[:, :rows], akc, odd)[0], _operand(B2, False, odd)[0]
        c = torch.zeros(rows, 150, dtype=torch.float64, device="cuda")
        pk.api.diag_gemm_forms(ta, tb, c, sa, (sb[1], sb[0], sb[2]), (150, 1, 0), rows, 150, K, 1,
                               A2=ta2 if two else None, B2=tb2 if two else None, ascending=True, splitk=True)
        got.append(c.cpu().numpy())
    f = 1.0 if two else 0.0
    size = np.abs(A[0]) @ np.abs(B[0].T) + f * np.abs(A2[0]) @ np.abs(B2[0].T)
    assert (np.abs(got[0] - A[0] @ B[0].T - f * A2[0] @ B2[0].T) <= 2 * (2 * K + 4) * 2.0 ** -53 * size).all()
    if K > 32:  # (shorter contractions of 20 rows have a kernel of their own)
        assert np.array_equal(got[0][:20], got[1])
