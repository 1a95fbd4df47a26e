"""FP64 products of more tiles than one row of a launch's grid holds, and
batches past the limit that every product shares."""

import pytest
import torch

import paper_2608_06669_amd as pk

pytestmark = pytest.mark.gpu


def test_more_tiles_than_one_grid_row_holds():
    """65535 products of 1 x 16448 x 40: 16842495 tiles, of which a row of
    256-thread workgroups takes fewer than 2^24; each output against the
    bound of any order of summation."""
    M, N, K, nb = 1, 16448, 40, 65535
    g = torch.Generator(device="cuda").manual_seed(5)
    a = torch.randn(nb, K, dtype=torch.float64, device="cuda", generator=g)
    b = torch.randn(N, K, dtype=torch.float64, device="cuda", generator=g)
    c = torch.full((nb, N), float("nan"), dtype=torch.float64, device="cuda")
    pk.api.diag_gemm_batched(a, b, c, (K, 1, K), (1, K, 0), (N, 1, N), M, N, K, nb)
    bound = 2 * (K + 3) * 2.0 ** -53
    for i in range(0, nb, 8192):
        x, y = a[i:i + 8192], c[i:i + 8192]
        ok = (y - x @ b.T).abs() <= bound * (x.abs() @ b.T.abs())
        assert bool(ok.all()), i


@pytest.mark.parametrize("K", [8, 40])
def test_batches_past_the_limit_are_refused(K):
    """Short contractions and long ones take different kernels, one limit."""
    a = torch.ones(K, dtype=torch.float64, device="cuda")
    c = torch.zeros(65536, dtype=torch.float64, device="cuda")
    with pytest.raises(pk.CCError):
        pk.api.diag_gemm_batched(a, a, c, (K, 1, 0), (1, K, 0), (1, 1, 1), 1, 1, K, 65536)
    pk.api.diag_gemm_batched(a, a, c, (K, 1, 0), (1, K, 0), (1, 1, 1), 1, 1, K, 65535)
    assert bool((c[:65535] == K).all()) and float(c[65535]) == 0.0
