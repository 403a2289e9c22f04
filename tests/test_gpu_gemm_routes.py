"""The two BF16 GEMM kernels (one wave per tile for short sums over many tiles, four
waves otherwise) do the same products in the same order: a wide product equals
its column blocks computed apart, bit for bit, on both sides of the lines."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(4096, 256, 96), (4080, 256, 96), (1029, 1030, 127), (1029, 1030, 128), (70000, 16, 5)])
@pytest.mark.parametrize("ta,tb", [(False, False), (True, False), (False, True), (True, True)])
def test_routes_agree(M, N, K, ta, tb):
    from paper_2410_04477_amd import api
    g = torch.Generator(device="cuda").manual_seed(M + K)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    A, B, bias, mask = r(M, K), r(K, N), r(N), r(M, N)
    op = lambda X, t: X.t().contiguous() if t else X
    for kw in (dict(bias=bias, relu=True), dict(mask=mask), dict(accumulate=True)):
        C0 = r(M, N)
        C = api.gemm(op(A, ta), op(B, tb), C0.clone(), ta=ta, tb=tb, **kw)
        want = torch.empty_like(C)
        for m0 in range(0, M, 2048):   # at most 2,080 tiles a call
            rows = slice(m0, min(M, m0 + 2048))
            for n0 in range(0, N, 256):
                cols = slice(n0, min(N, n0 + 256))
                sub = {k: (v[cols].contiguous() if k == "bias" else v[rows, cols].contiguous() if k == "mask" else v)
                       for k, v in kw.items()}
                want[rows, cols] = api.gemm(op(A[rows].contiguous(), ta), op(B[:, cols].contiguous(), tb),
                                            C0[rows, cols].contiguous(), ta=ta, tb=tb, **sub)
        assert torch.equal(C, want)
    ref = A.bfloat16().double() @ B.bfloat16().double()
    got = api.gemm(op(A, ta), op(B, tb), torch.empty_like(C), ta=ta, tb=tb)
    # FP32 sums of K terms: K 2^-24 of the sum of magnitudes, doubled
    bound = 2 * K * 2.0 ** -24 * (A.bfloat16().double().abs() @ B.bfloat16().double().abs())
    assert bool(((got.double() - ref).abs() <= bound).all())
