"""The output of the four-wave GEMM kernel straight from its registers (rp_op_gemm tile 7): at the edges of its 16-row, 32-column and 256-wide
units, against the eight-wave kernel (tile 1), which stages its tile through LDS -- the same reduction, so the same bits -- and
with everything around the output left alone."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SHAPES = [(1, 8), (17, 72), (129, 136), (255, 264), (272, 520), (513, 248)]


@pytest.mark.parametrize("layout", (0, 1, 2))
@pytest.mark.parametrize("out", ("bf16", "residual", "fp32", "fp32 +="))
def test_rows_from_registers(layout, out):
    from paper_2604_27085_amd import binding as B
    torch.manual_seed(5)
    dev = "cuda:0"
    st = torch.cuda.current_stream().cuda_stream
    for M, N in SHAPES:
        if layout == 2:
            M = (M + 7) // 8 * 8
        for K, alpha in ((64, 1.0), (200, 0.37)):
            bf = lambda *s: torch.randn(*s, device=dev).to(torch.bfloat16)  # noqa: E731
            A = bf(K, M) if layout == 2 else bf(M, K)
            W = bf(N, K) if layout == 0 else bf(K, N)
            R = bf(M, N + 4) if out == "residual" else None
            ldc = N + 8
            start = torch.full((M + 3, ldc), 7.0, dtype=torch.float32 if out[0] == "f" else torch.bfloat16, device=dev)
            got = []
            for tile in (1, 7):
                C = start.clone()
                B.rp_op_gemm(st, layout, int(out[0] == "f"), A, W, C, M, N, K, A.shape[1], W.shape[1], ldc, alpha, int(out == "fp32 +="), R=R,
                             ldr=N + 4, tile=tile)
                got.append(C)
            torch.cuda.synchronize()
            assert torch.equal(got[0], got[1]), (M, N, K)
            assert bool((got[1][M:] == 7.0).all()) and bool((got[1][:, N:] == 7.0).all()), (M, N, K)
            exact = alpha * ((A.double().t() if layout == 2 else A.double()) @ (W.double().t() if layout == 0 else W.double()))
            if R is not None:
                exact = exact + R[:, :N].double()
            if out == "fp32 +=":
                exact = exact + 7.0
            # one rounding to bf16 (2^-9), or fp32 sums of K products
            assert float((got[1][:M, :N].double() - exact).norm() / exact.norm()) < (2.0 ** -8 if out[0] != "f" else 1e-6)
