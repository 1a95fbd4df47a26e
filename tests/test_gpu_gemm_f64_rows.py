"""FP64 products of operands whose rows are far apart (2^22 elements and more,
as the contraction over (l, c, d) of o v^2 >= 2^22 has) or stored backwards."""

import numpy as np
import pytest
import torch

import paper_2608_06669_amd as pk

pytestmark = pytest.mark.gpu


def _place(x, kc, ld):
    """x [rows][K] with rows (kc) or columns ld elements apart, the last one
    first if ld < 0. Returns (view from its first element, strides of row and
    k)."""
    y = torch.tensor(np.ascontiguousarray(x if kc else x.T), device="cuda")
    buf = torch.zeros((y.shape[0] - 1) * abs(ld) + y.shape[1], dtype=torch.float64, device="cuda")
    view = torch.as_strided(buf, y.shape, (abs(ld), 1))
    view.copy_(y if ld > 0 else y.flip(0))
    first = buf if ld > 0 else buf[(y.shape[0] - 1) * -ld:]
    return first, (ld if kc else 1), (1 if kc else ld)


@pytest.mark.parametrize("M,N,K", [(70, 66, 39), (20, 36, 1001)])
@pytest.mark.parametrize("akc,bkc", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("ld", [2 ** 22, 2 ** 22 + 1, -1002])
def test_rows_far_apart_take_the_same_kernel(M, N, K, akc, bkc, ld):
    """The same sums in the same order as for short rows, bit for bit (a kernel
    with another order of k differs in the last bits of most elements), within
    the bound of any order of summation."""
    if abs(ld) >= 2 ** 22 and not (akc and bkc):
        K = min(K, 39)  # (K rows of 32 MB)
    rng = np.random.default_rng(M + N + K)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((N, K))
    got = []
    for stride in (ld, 1002 + ld % 2):  # (of the same alignment)
        (ta, a_r, a_k), (tb, b_r, b_k) = _place(A, akc, stride), _place(B, bkc, stride)
        tc = torch.zeros(M, N, dtype=torch.float64, device="cuda")
        pk.api.diag_gemm_batched(ta, tb, tc, (a_r, a_k, 0), (b_k, b_r, 0), (N, 1, 0), M, N, K, 1, splitk=True)
        got.append(tc.cpu().numpy())
    size = np.abs(A) @ np.abs(B.T)
    assert (np.abs(got[0] - A @ B.T) <= 2 * (K + 3) * 2.0 ** -53 * size).all()
    assert np.array_equal(got[0], got[1])
