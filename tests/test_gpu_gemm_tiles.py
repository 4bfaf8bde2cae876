"""Small-tile GEMMs (operands loaded straight into LDS, waves of 64x64) at the edges of their tiles, and the stage calls whose
products they serve.  bf16 results: one rounding of an fp32 sum, relative error 2^-9 = 2e-3, bound 4e-3; fp32 results: sums of
at most 1300 products of bf16 values in fp32, bound 1e-5."""
import numpy as np
import pytest

import parity_util as pu
import synth
from test_gpu_kernels import dev, rel_l2, rnd, stream

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding, harness
    return binding, harness


# (M, N, K, K2): one element past and one short of 64, 128 and 256; K of one tile, of fewer tiles than there are wave groups,
# with a tail; a second operand pair shorter and longer than a K tile; skinny outputs; a reduction long enough to be split
SHAPES = [(8, 8, 8, 0), (64, 64, 64, 0), (72, 56, 192, 0), (120, 136, 136, 24), (264, 248, 72, 8), (136, 520, 328, 72), (1016, 16, 1288, 0),
          (48, 1032, 1160, 16), (200, 128, 1304, 40)]


@pytest.mark.parametrize("tile", [0, 2, 3, 4])
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_small_tiles_at_their_edges(rp, layout, tile):
    B, H = rp
    for M, N, K, K2 in SHAPES:
        rng = np.random.default_rng(9000 + M + N + K)
        a, b, res = rnd(rng, (M, K)), rnd(rng, (N, K), 0.05), rnd(rng, (M, N))
        u, v = rnd(rng, (M, max(K2, 8))), rnd(rng, (N, max(K2, 8)), 0.1)
        ref = a.astype(np.float64) @ b.T.astype(np.float64)
        if K2:
            ref += u.astype(np.float64) @ v.T.astype(np.float64)
        t = lambda m, swap: dev(H, np.ascontiguousarray(m.T) if swap else m)  # noqa: E731
        A, Bm, lda, ldb = t(a, layout == 2), t(b, layout > 0), M if layout == 2 else K, K if layout == 0 else N
        kw = dict(tile=tile)
        if K2:
            kw.update(A2=t(u, layout == 2), B2=t(v, layout > 0), K2=K2, lda2=M if layout == 2 else K2, ldb2=K2 if layout == 0 else N)
        ws = torch.full((16 * M * N,), float("nan"), dtype=torch.float32, device="cuda:0")
        R = dev(H, res)
        outs = []
        for split in (None, ws, ws):      # with scratch the product may be cut along the reduction: same result, twice the same bits
            C16 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
            B.rp_op_gemm(stream(), layout, 0, A, Bm, C16, M, N, K, lda, ldb, N, alpha=-0.5, R=R, ldr=N, split_ws=split, **kw)
            C32 = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda:0")
            B.rp_op_gemm(stream(), layout, 1, A, Bm, C32, M, N, K, lda, ldb, N, alpha=0.5, beta=1, split_ws=split, **kw)
            torch.cuda.synchronize()
            assert rel_l2(H.to_f32(C16), -0.5 * ref + res) < 4e-3, (M, N, K, K2)
            assert rel_l2(C32.cpu().numpy(), 0.5 * ref + 2.0) < 1e-5, (M, N, K, K2)
            outs.append((C16, C32))
        assert torch.equal(outs[1][0], outs[2][0]) and torch.equal(outs[1][1], outs[2][1])
        Ca = torch.full((M, N), 1.0, dtype=torch.float32, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 2, A, Bm, Ca, M, N, K, lda, ldb, N, **kw)
        torch.cuda.synchronize()
        assert rel_l2(Ca.cpu().numpy(), ref + 1.0) < 1e-5, (M, N, K, K2)


@pytest.mark.parametrize("seq,batch,ffn,hidden", [(8, 1, 384, 256), (36, 2, 64, 256), (136, 1, 328, 256), (264, 1, 72, 256),
                                                  (1040, 1, 4680, 512), (520, 1, 8264, 2560)])
def test_short_stage_with_swiglu_epilogues(rp, seq, batch, ffn, hidden):
    """The SwiGLU forward and backward ride in the epilogues of the small tiles, and of the two 256x256 kernels in the last
    two (reductions of 512 and 2560); gate and up columns that end inside a tile; adapters on all projections."""
    c = synth.shrink(synth.CONFIGS["C1"], n_layers=1, hidden=hidden, ffn=ffn, vocab=0, seq=seq, batch=batch, lora=synth.LORA_ORDER,
                     x_from="normal")
    wl = synth.make_workload(c, 4242 + seq, gains_random=True)
    errs = pu.compare_chain(pu.oracle_chain(c, wl, dtype=np.float32), pu.gpu_chain(c, wl, rp[1]), c)
    assert max(errs.values()) <= 2e-2
