"""Small-tile GEMMs (operands loaded straight into LDS, waves of 64x64) at the edges of their tiles, and the stage calls whose
products they serve.  bf16 results: one rounding of an fp32 sum, relative error 2^-9 = 2e-3, bound 4e-3; fp32 results: a
sum of n products in fp32 is off by at most about sqrt(n) 2^-24 of its size when the errors are independent, 7e-6 for the longest
reduction here (12320), bound 1e-5."""
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
    """The SwiGLU forward and backward ride in the epilogues of the small tiles, the forward of the last two (reductions of 512 and 2560) in that
    of the four-wave 256x256 kernel; gate and up columns that end inside a tile; adapters on all projections."""
    c = synth.shrink(synth.CONFIGS["C1"], n_layers=1, hidden=hidden, ffn=ffn, vocab=0, seq=seq, batch=batch, lora=synth.LORA_ORDER,
                     x_from="normal")
    wl = synth.make_workload(c, 4242 + seq, gains_random=True)
    errs = pu.compare_chain(pu.oracle_chain(c, wl, dtype=np.float32), pu.gpu_chain(c, wl, rp[1]), c)
    assert max(errs.values()) <= 2e-2


@pytest.mark.parametrize("hidden", [256, 512])
def test_swiglu_epilogues_of_the_256x256_tiles(rp, hidden):
    """Forward (408 tiles) and backward (208) on 256x256 tiles that end inside a tile in both directions: reductions of 256 run the eight-wave
    kernel, whose tiles go out through LDS, those of 512 the four-wave one, straight from the registers."""
    B, H = rp
    T, m = 2040, 6408
    c = synth.shrink(synth.CONFIGS["C1"], n_layers=1, hidden=hidden, ffn=m, vocab=0, seq=T, batch=1, lora_rank=0, lora=(), x_from="normal")
    wl = synth.make_workload(c, 4300 + hidden, gains_random=True)
    errs = pu.compare_chain(pu.oracle_chain(c, wl, dtype=np.float32), pu.gpu_chain(c, wl, H), c)
    assert max(errs.values()) <= 2e-2
    r = H.StageRunner(H.cfg_from_dict(c), 1, T)      # and those tiles they were
    try:
        r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
        x = torch.empty((T, hidden), dtype=torch.bfloat16, device="cuda:0").normal_()
        dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
        torch.cuda.synchronize()
        r.bind()
        B.rp_trace_start(r.ctx, 256)
        B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, r.grads, None, None, 1, T, r.ws, r.wsbytes)
        rec = B.rp_trace_stop(r.ctx, 256)
    finally:
        r.close()
    product = 2.0 * T * hidden * m
    assert [t[0] for t in rec if t[1] == 2 * product and t[0].endswith("NT")] == ["gemm_256x256_NT"]
    assert [t[0] for t in rec if t[1] == product and t[0].endswith("NN")] == ["gemm_256x256_NN"]


def operand(rng, rows, cols, std=1.0):
    """bf16 [rows, cols] on the GPU, drawn there."""
    return torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=rng)


def product(rng, layout, M, N, K, K2):
    """Operands of one product as the layout stores them, their leading dimensions, and the product in 64 bits."""
    kw, ref = {}, 0.0
    for x, y, k, sfx in ((("A", "B", K, ""), ("A2", "B2", K2, "2")) if K2 else (("A", "B", K, ""),)):
        a, b = operand(rng, M, k), operand(rng, N, k, 0.05)
        ref = ref + a.double() @ b.double().t().contiguous()
        kw[x], kw["lda" + sfx] = (a.t().contiguous(), M) if layout == 2 else (a, k)
        kw[y], kw["ldb" + sfx] = (b.t().contiguous(), N) if layout else (b, k)
    return kw, ref


def err(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


# (M, N, K, K2) that the cost model cuts along the reduction, with the tile it takes: 256x256 (four waves), 128x128, 128x64, 128x128 with
# eight rows, 128x64 (two), 64x64 (three), 256x128 by two groups
SPLIT_SHAPES = [(1032, 2056, 12296, 24), (1016, 1032, 8200, 24), (520, 1032, 4104, 24), (8, 2056, 4104, 16), (72, 72, 1288, 24),
                (1032, 136, 2312, 24), (136, 56, 1288, 0), (8, 264, 4104, 8), (8, 8, 12296, 0), (1544, 520, 12296, 24)]


@pytest.mark.parametrize("shape", SPLIT_SHAPES)
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_automatic_splits_of_the_reduction(rp, layout, shape):
    """The product really is cut (the slices' partial products, and nothing behind them, replace what the scratch held), the merge
    takes the residual or the old value, and the sum does not depend on the run; scratch that holds one slice is left alone."""
    B, _ = rp
    M, N, K, K2 = shape
    rng = torch.Generator(device="cuda:0").manual_seed(M + N + K + layout)
    kw, ref = product(rng, layout, M, N, K, K2)
    A, Bm, lda, ldb = (kw.pop(k) for k in ("A", "B", "lda", "ldb"))
    if K2:
        kw["K2"] = K2
    R = operand(rng, M, N)
    for f32, want, bound in ((0, -0.5 * ref + R.double(), 4e-3), (1, 0.5 * ref + 2.0, 1e-5)):
        outs = []
        for ws in (torch.full((16 * M * N + 64,), float("nan"), device="cuda:0"), torch.full((16 * M * N + 64,), float("nan"), device="cuda:0"),
                   torch.full((M * N,), float("nan"), device="cuda:0")):
            C = torch.full((M, N), 2.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda:0")
            if f32:
                B.rp_op_gemm(stream(), layout, 1, A, Bm, C, M, N, K, lda, ldb, N, alpha=0.5, beta=1, split_ws=ws, **kw)
            else:
                B.rp_op_gemm(stream(), layout, 0, A, Bm, C, M, N, K, lda, ldb, N, alpha=-0.5, R=R, ldr=N, split_ws=ws, **kw)
            torch.cuda.synchronize()
            assert err(C, want) < bound
            outs.append(C)
            written = int((~torch.isnan(ws)).sum())
            if ws.numel() == M * N:
                assert written == 0
            else:
                assert written % (M * N) == 0 and 2 <= written // (M * N) <= 16 and not torch.isnan(ws[:written]).any()
        assert torch.equal(outs[0], outs[1])


# (layout, fp32 output, accumulate, M, N, K, K2, residual): what the adapters of a projection are made of; long and short reductions;
# one that does not share the launch (561 tiles of 64x64)
GROUP = [(1, 0, 0, 1016, 16, 4104, 0, 0), (2, 1, 1, 4104, 16, 1016, 0, 0), (2, 1, 1, 72, 520, 1016, 0, 0), (0, 0, 0, 264, 136, 2568, 24, 1),
         (1, 0, 0, 1032, 2056, 264, 0, 0), (0, 1, 0, 8, 8, 8, 0, 0), (2, 1, 1, 136, 56, 12296, 0, 0), (1, 0, 0, 48, 1032, 328, 40, 1)]


@pytest.mark.parametrize("scratch", ["none", "one product's three slices", "all"])
@pytest.mark.parametrize("members", [(0, 1, 2, 3, 4, 5, 6, 7), (6, 3), (4, 5), (4,), (0, 1, 2)])
def test_products_that_share_a_launch(rp, members, scratch):
    B, _ = rp
    floats = {"none": 0, "one product's three slices": 3 * 1016 * 16 + 8, "all": sum(16 * GROUP[i][3] * GROUP[i][4] for i in members)}[scratch]
    runs = []
    for _ in range(2):
        rng = torch.Generator(device="cuda:0").manual_seed(77)
        descs, checks = [], []
        for i in members:
            layout, f32, beta, M, N, K, K2, res = GROUP[i]
            d, ref = product(rng, layout, M, N, K, K2)
            C = torch.full((M, N + 8), 3.0, dtype=torch.float32 if f32 else torch.bfloat16, device="cuda:0")    # rows with room behind them
            R = operand(rng, M, N) if res else None
            d.update(C=C, ldc=N + 8, layout=layout, out_f32=f32, M=M, N=N, K=K, K2=K2, beta=beta, alpha=0.5)
            if res:
                d.update(R=R, ldr=N)
            descs.append(d)
            checks.append((i, C, 0.5 * ref + (R.double() if res else 0.0) + (3.0 if beta else 0.0), 1e-5 if f32 else 4e-3))
        ws = torch.full((floats,), float("nan"), device="cuda:0") if floats else None
        torch.cuda.synchronize()
        B.rp_op_gemm_group(stream(), descs, split_ws=ws)
        torch.cuda.synchronize()
        for i, C, want, bound in checks:
            N = GROUP[i][4]
            assert err(C[:, :N], want) < bound, GROUP[i]
            assert bool((C[:, N:] == 3.0).all()), GROUP[i]
        runs.append([C for _, C, _, _ in checks])
        if ws is not None and members in ((0, 1, 2, 3, 4, 5, 6, 7), (0, 1, 2)):      # the first product is cut, into slices of [1016, 16]
            assert not torch.isnan(ws[:2 * 1016 * 16]).any()
    assert all(torch.equal(a, b) for a, b in zip(*runs))


def test_a_group_refuses_what_a_single_product_refuses(rp):
    B, _ = rp
    a = torch.zeros((64, 64), dtype=torch.bfloat16, device="cuda:0")
    ok = dict(A=a, B=a, C=a, lda=64, ldb=64, ldc=64, layout=0, M=64, N=64, K=64)
    for bad in (dict(A=None), dict(K=12), dict(lda=60), dict(layout=3), dict(out_f32=2), dict(M=-1)):
        with pytest.raises(B.RpError) as e:
            B.rp_op_gemm_group(stream(), [ok, dict(ok, **bad)])
        assert e.value.code == B.RP_EINVAL
    with pytest.raises(B.RpError):
        B.rp_op_gemm_group(stream(), [ok] * 9)


@pytest.mark.parametrize("tile", [0, 2, 3, 4])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("K2", [0, 24, 136])
def test_small_tiles_with_an_empty_first_pair(rp, layout, tile, K2):
    """K = 0: the reduction is the second operand pair alone, or nothing (then the result is the residual, or the old value)."""
    B, _ = rp
    M, N = 136, 72
    rng = torch.Generator(device="cuda:0").manual_seed(K2)
    kw, ref = product(rng, layout, M, N, max(K2, 8), 0)
    ref = ref if K2 else torch.zeros_like(ref)
    X, Y, ldx, ldy = (kw.pop(k) for k in ("A", "B", "lda", "ldb"))
    pair = dict(A2=X, B2=Y, K2=K2, lda2=ldx, ldb2=ldy) if K2 else {}
    R = operand(rng, M, N)
    for split in (None, torch.full((16 * M * N,), float("nan"), device="cuda:0")):
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 0, X, Y, C, M, N, 0, ldx, ldy, N, R=R, ldr=N, tile=tile, split_ws=split, **pair)
        C32 = torch.full((M, N), 2.0, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 1, X, Y, C32, M, N, 0, ldx, ldy, N, beta=1, tile=tile, split_ws=split, **pair)
        torch.cuda.synchronize()
        assert err(C, ref + R.double()) < 4e-3 and err(C32, ref + 2.0) < 1e-5
        if not K2:
            assert torch.equal(C, R) and bool((C32 == 2.0).all())
