"""FP32 / BF16 products with few rows or columns (one or two 16-row tiles,
either operand layout, ragged edges, short and split contractions, batches,
operands rounded on load or beforehand) against FP64 products of the rounded
operands. FP32 accumulation of K products errs by at most (K + 2) 2^-23 of
sum |a b|; the bound here is that, elementwise."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1, 1, 1), (1, 3001, 60, 1), (16, 33, 32, 3), (17, 40, 33, 2), (32, 70, 129, 1), (20, 1000, 20, 4),
          (33, 31, 64, 1), (300, 20, 77, 2), (2050, 1, 515, 1), (20, 180, 20000, 1)]


@pytest.mark.parametrize("M,N,K,nb", SHAPES)
@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_thin_product(M, N, K, nb, ta, tb, prec):
    import paper_2608_06669_amd as pk
    g = torch.Generator(device="cpu").manual_seed(M + 10 * N + K)
    A = torch.randn(nb, K if ta else M, M if ta else K, generator=g, dtype=torch.float64)
    B = torch.randn(nb, N if tb else K, K if tb else N, generator=g, dtype=torch.float64)
    C = torch.randn(nb, M, N, generator=g, dtype=torch.float64)
    low = torch.float32 if prec == "fp32" else torch.bfloat16
    a, b = ((x.float().to(low).double().transpose(1, 2) if t else x.float().to(low).double()) for x, t in ((A, ta), (B, tb)))
    want = torch.stack([0.5 * x @ y for x, y in zip(a, b)]) - 2.0 * C
    bound = (K + 2) * 2.0 ** -23 * torch.stack([0.5 * x.abs() @ y.abs() for x, y in zip(a, b)]) + 1e-14 * C.abs() + 1e-14
    for precast, splitk in [(False, False), (False, True), (True, True)]:
        Cd = C.cuda()
        pk.diag_gemm_batched(A.cuda(), B.cuda(), Cd, (1, M, M * K) if ta else (K, 1, M * K),
                             (1, K, N * K) if tb else (N, 1, N * K), (N, 1, M * N), M, N, K, nb, alpha=0.5, beta=-2.0,
                             prec=prec, precast=precast, splitk=splitk)
        torch.cuda.synchronize()
        assert bool(((Cd.cpu() - want).abs() <= bound).all())


@pytest.mark.parametrize("M,N,K", [(2049, 2047, 4), (2048, 2048, 32), (2049, 2047, 36), (2050, 2113, 100), (2049, 2047, 1028)])
def test_wide_fp32_product(M, N, K):
    """FP32 products in one piece with both operands rounded beforehand: ragged
    128 x 64 tiles, one to 33 panels of 32 with and without a remainder."""
    import paper_2608_06669_amd as pk
    g = torch.Generator(device="cpu").manual_seed(K)
    A = torch.randn(M, K, generator=g, dtype=torch.float64)
    B = torch.randn(K, N, generator=g, dtype=torch.float64)
    C = torch.randn(M, N, generator=g, dtype=torch.float64)
    a, b = A.float().double(), B.float().double()
    want = 0.5 * a @ b - 2.0 * C
    bound = (K + 2) * 2.0 ** -23 * (0.5 * a.abs() @ b.abs()) + 1e-14 * C.abs() + 1e-14
    Cd = C.cuda()
    pk.diag_gemm_batched(A.cuda(), B.cuda(), Cd, (K, 1, 0), (N, 1, 0), (N, 1, 0), M, N, K, 1, alpha=0.5, beta=-2.0,
                         prec="fp32", precast=True, splitk=True)
    torch.cuda.synchronize()
    assert bool(((Cd.cpu() - want).abs() <= bound).all())
