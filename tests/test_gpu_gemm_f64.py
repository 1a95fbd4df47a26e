"""The FP64 product at the edges of its tiles, panels and chunks, for every
operand layout it takes, against numpy's float64 product (the bound is that of
any summation order: (K + 3) 2^-53 times the sum of the terms' sizes)."""

import numpy as np
import pytest
import torch

import paper_2608_06669_amd as pk

pytestmark = pytest.mark.gpu


def _operand(x, kc, ld, base):
    """The batch x [nb][rows][K] in device memory of row length `ld`, its
    first element `base` doubles into the allocation; what lies between the
    rows is NaN. Returns (tensor view, stride of rows, of k, of the batch)."""
    nb, rows, K = x.shape
    y = x if kc else x.transpose(0, 2, 1)
    buf = np.full((nb, y.shape[1], ld), np.nan)
    buf[:, :, : y.shape[2]] = y
    t = torch.tensor(np.concatenate([np.full(base, np.nan), buf.ravel()]), device="cuda")[base:]
    return t, (ld if kc else 1), (1 if kc else ld), y.shape[1] * ld


# (M, N, K, nbatch, splitk): one tile and less, the edges of 64-row tiles and
# 8-deep panels, 1 to 9 panels (the loop takes them four at a time), remainders
# of one and seven columns, whole rounds of 256 tiles with a cut tail, few
# tiles with many chunks, and a product large enough for 128-column tiles
SIZES = [(1, 1, 1, 1, False), (3, 70, 8, 1, False), (64, 64, 16, 2, False), (65, 66, 24, 1, False),
         (66, 64, 32, 3, False), (63, 65, 33, 1, False), (130, 62, 39, 1, False), (128, 192, 72, 1, False),
         (1100, 1090, 96, 1, True), (70, 66, 1001, 1, True), (2, 2, 5000, 2, True), (20, 18, 40000, 1, True),
         (130, 8190, 9802, 1, True),
         # rows that tiles of 48, 72 and 80 fit
         (48, 130, 40, 2, False), (143, 66, 100, 1, True), (79, 129, 1001, 1, True), (150, 200, 64, 1, False)]


@pytest.mark.parametrize("M,N,K,nb,splitk", SIZES)
@pytest.mark.parametrize("akc,bkc", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("even", [True, False], ids=["aligned", "unaligned"])
def test_f64_product_at_the_edges(M, N, K, nb, splitk, akc, bkc, even):
    rng = np.random.default_rng(M * 7 + N * 5 + K)
    A = rng.standard_normal((nb, M, K))
    B = rng.standard_normal((nb, N, K))
    C0 = rng.standard_normal((nb, M, N))
    # rows of even length on 16-byte boundaries, or odd ones one element off
    length = lambda n: n + 2 + (n % 2 if even else 1 - n % 2)  # noqa: E731
    base = 0 if even else 1
    ta, a_r, a_k, a_b = _operand(A, akc, length(K if akc else M), base)
    tb, b_r, b_k, b_b = _operand(B, bkc, length(K if bkc else N), base)
    tc = torch.tensor(C0, device="cuda")
    pk.api.diag_gemm_batched(ta, tb, tc, (a_r, a_k, a_b), (b_k, b_r, b_b), (N, 1, M * N), M, N, K, nb, alpha=-0.5,
                             beta=2.0, splitk=splitk)
    ref = -0.5 * np.matmul(A, B.transpose(0, 2, 1)) + 2.0 * C0
    size = 0.5 * np.matmul(np.abs(A), np.abs(B.transpose(0, 2, 1))) + 2.0 * np.abs(C0)
    err = np.abs(tc.cpu().numpy() - ref)
    assert (err <= 2 * (K + 3) * 2.0 ** -53 * size).all(), float((err / size).max())


def test_f64_product_of_operands_contiguous_along_neither_index():
    rng = np.random.default_rng(3)
    M, N, K = 70, 65, 19
    a = torch.tensor(rng.standard_normal((2 * M, 3 * K)), device="cuda")
    b = torch.tensor(rng.standard_normal((2 * N, 2 * K)), device="cuda")
    c = torch.zeros(M, N, dtype=torch.float64, device="cuda")
    pk.api.diag_gemm(a, b, c, (6 * K, 3), (2, 4 * K), (N, 1), M, N, K)
    x, y = a.cpu().numpy()[::2, ::3], b.cpu().numpy()[::2, ::2]
    ref, size = x @ y.T, np.abs(x) @ np.abs(y.T)
    assert (np.abs(c.cpu().numpy() - ref) <= 2 * (K + 3) * 2.0 ** -53 * size).all()
