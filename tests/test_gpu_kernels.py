"""Kernel-by-kernel parity of the HIP library (through its C ABI) against the CPU oracle, on seeded inputs at sizes that
span several tiles and a ragged tail.  Tolerance: relative L2 error <= 2e-2 for bf16 results (the bound the task
states), much tighter where the result is fp32."""
import numpy as np
import pytest

import synth
from oracle import layers as L

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding, harness
    return binding, harness


def rel_l2(a, b):
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def rnd(rng, shape, std=1.0):
    return synth.bf16_round(rng.standard_normal(shape, dtype=np.float32) * np.float32(std))


def dev(h, arr):
    return h.bf16_tensor(arr, "cuda:0")


def stream():
    return torch.cuda.current_stream().cuda_stream


# ----------------------------------------------------------------------------------------------- GEMM
@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("layout", [0, 1, 2])
def test_gemm_layouts_ragged(rp, layout, tile):
    B, H = rp
    rng = np.random.default_rng(100 + layout * 10 + tile)
    M, N, K = 328, 264, 200          # ragged against every tile size, K not a multiple of 64
    a = rnd(rng, (M, K))
    b = rnd(rng, (N, K))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    if layout == 0:
        A, Bm, lda, ldb = dev(H, a), dev(H, b), K, K
    elif layout == 1:
        A, Bm, lda, ldb = dev(H, a), dev(H, np.ascontiguousarray(b.T)), K, N
    else:
        A, Bm, lda, ldb = dev(H, np.ascontiguousarray(a.T)), dev(H, np.ascontiguousarray(b.T)), M, N
    Cm = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_gemm(stream(), layout, 0, A, Bm, Cm, M, N, K, lda, ldb, N, tile=tile)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(Cm), ref) < 4e-3
    # fp32 output, accumulate on top of an existing value, alpha
    C32 = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda:0")
    B.rp_op_gemm(stream(), layout, 1, A, Bm, C32, M, N, K, lda, ldb, N, alpha=0.25, beta=1, tile=tile)
    torch.cuda.synchronize()
    assert rel_l2(C32.cpu().numpy(), 0.25 * ref + 0.5) < 1e-5
    # fp32 output that overwrites what the buffer held (no accumulation, unit scale)
    C32.fill_(float("nan"))
    B.rp_op_gemm(stream(), layout, 1, A, Bm, C32, M, N, K, lda, ldb, N, beta=0, tile=tile)
    torch.cuda.synchronize()
    assert rel_l2(C32.cpu().numpy(), ref) < 1e-5
    # bf16 output with a scale
    Cm.fill_(float("nan"))
    B.rp_op_gemm(stream(), layout, 0, A, Bm, Cm, M, N, K, lda, ldb, N, alpha=-0.5, tile=tile)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(Cm), -0.5 * ref) < 4e-3


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("shape", [(584, 456, 712, 40), (256, 256, 64, 0), (1, 8, 8, 16), (700, 1032, 2056, 0), (300, 520, 0, 24)])
def test_gemm_operands_loaded_straight_into_lds(rp, shape, layout):
    """Tile 7 (what tile 0 picks on 256x256 tiles when the reduction is long): four waves of 128x128, operands fetched from memory
    straight into a ring of LDS units, reduction tails and tiles past the end read through out-of-range offsets.
    Against the fp64 product, and bit for bit against the staged eight-wave kernel (tile 1: a wider matrix instruction,
    same order of the reduction).  Ragged rows and columns against 256/128/64, K and K2 against the K tile of 64 (the
    second pair shorter than one tile, a first pair of one tile exactly, an empty first pair); residual, fp32
    accumulation with alpha, a reduction split merged in slice order."""
    B, H = rp
    M, N, K, K2 = shape
    rng = np.random.default_rng(700 + M + K)
    a, b = rnd(rng, (M, max(K, 8))), rnd(rng, (N, max(K, 8)), 0.05)
    u, bl = rnd(rng, (M, max(K2, 8))), rnd(rng, (N, max(K2, 8)), 0.1)
    res = rnd(rng, (M, N))
    ref = a[:, :K].astype(np.float64) @ b[:, :K].T.astype(np.float64) + u[:, :K2].astype(np.float64) @ bl[:, :K2].T.astype(np.float64)
    if layout == 2:      # A [K, M]: rows of A have to come in multiples of 8
        M = (M + 7) // 8 * 8
        a, u, res = rnd(rng, (M, max(K, 8))), rnd(rng, (M, max(K2, 8))), rnd(rng, (M, N))
        ref = a[:, :K].astype(np.float64) @ b[:, :K].T.astype(np.float64) + u[:, :K2].astype(np.float64) @ bl[:, :K2].T.astype(np.float64)
        A, A2, R = dev(H, np.ascontiguousarray(a.T)), dev(H, np.ascontiguousarray(u.T)), dev(H, res)
        lda, lda2 = M, M
    else:
        A, A2, R = dev(H, a), dev(H, u), dev(H, res)
        lda, lda2 = max(K, 8), max(K2, 8)
    if layout == 0:      # B [N, K], reduction index contiguous
        Bm, ldb, B2m, ldb2 = dev(H, b), max(K, 8), dev(H, bl), max(K2, 8)
    else:                # B [K, N]: read with the transposing LDS load
        Bm, ldb, B2m, ldb2 = dev(H, np.ascontiguousarray(b.T)), N, dev(H, np.ascontiguousarray(bl.T)), N
    kw = dict(A2=A2, B2=B2m, K2=K2, lda2=lda2, ldb2=ldb2) if K2 else {}
    ws = torch.empty(16 * M * N, dtype=torch.float32, device="cuda:0")
    outs = []
    for tile in (1, 7):
        Cm = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 0, A, Bm, Cm, M, N, K, lda, ldb, N, R=R, ldr=N, tile=tile, **kw)
        C32 = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 1, A, Bm, C32, M, N, K, lda, ldb, N, alpha=0.25, beta=1, tile=tile, **kw)
        Cs = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda:0")     # with scratch: may be cut along the reduction
        B.rp_op_gemm(stream(), layout, 1, A, Bm, Cs, M, N, K, lda, ldb, N, beta=1, tile=tile, split_ws=ws, **kw)
        torch.cuda.synchronize()
        outs.append((H.to_f32(Cm), C32.cpu().numpy(), Cs.cpu().numpy()))
    scale = max(np.sqrt(np.mean(ref ** 2)), 1e-3)
    assert np.sqrt(np.mean((outs[1][0] - (ref + res)) ** 2)) < 4e-3 * max(scale, np.sqrt(np.mean((ref + res) ** 2)))
    assert np.sqrt(np.mean((outs[1][1] - (0.25 * ref + 0.5)) ** 2)) < 1e-5 * (scale + 0.5)
    assert np.sqrt(np.mean((outs[1][2] - (ref + 0.5)) ** 2)) < 1e-5 * (scale + 0.5)
    for got, want in zip(outs[1], outs[0]):
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("M,N,K", [(300, 520, 2624), (256, 264, 64), (1, 8, 2560)])
def test_gemm_residual_with_rows_on_8_byte_boundaries(rp, M, N, K):
    """The residual's row stride is a multiple of 4 only, and its rows start 8 bytes off a 16-byte boundary: the four-wave kernel, which
    reads it ahead in rows of 64 columns, against the eight-wave kernel bit for bit and against the fp64 product."""
    B, H = rp
    rng = np.random.default_rng(800 + M)
    a, b, res = rnd(rng, (M, K)), rnd(rng, (N, K), 0.05), rnd(rng, (M, N))
    ldr = N + 4
    R = torch.full((M * ldr + 4,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    R[4:].view(M, ldr)[:, :N] = dev(H, res)
    A, Bm = dev(H, a), dev(H, b)
    outs = []
    for tile in (1, 7):
        Cm = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        torch.cuda.synchronize()
        B.rp_op_gemm(stream(), 0, 0, A, Bm, Cm, M, N, K, K, K, N, R=R[4:], ldr=ldr, tile=tile)
        torch.cuda.synchronize()
        outs.append(H.to_f32(Cm))
    ref = a.astype(np.float64) @ b.T.astype(np.float64) + res
    assert rel_l2(outs[1], ref) < 4e-3
    np.testing.assert_array_equal(outs[0], outs[1])


@pytest.mark.parametrize("layout", [0, 1])
def test_gemm_b_operand_in_fragment_order(rp, layout):
    """Tile 6: B (and the second pair's B) pre-arranged in the fragment order of the matrix instruction and streamed
    into registers without LDS.  Against the fp64 product, and bit for bit against the staged 256x256 kernel (same
    operand values, same order of multiply-adds).  Ragged everywhere: rows and columns against 256/64, K and K2 against
    the K tile of 64; second operand pair, residual, fp32 accumulation."""
    B, H = rp
    rng = np.random.default_rng(300 + layout)
    M, N, K, K2 = 584, 456, 712, 40
    a, b = rnd(rng, (M, K)), rnd(rng, (N, K), 0.05)
    u, bl = rnd(rng, (M, K2)), rnd(rng, (N, K2), 0.1)
    res = rnd(rng, (M, N))
    ref = a.astype(np.float64) @ b.T.astype(np.float64) + u.astype(np.float64) @ bl.T.astype(np.float64)
    if layout == 0:
        Bm, ldb, B2m, ldb2 = dev(H, b), K, dev(H, bl), K2
    else:
        Bm, ldb, B2m, ldb2 = dev(H, np.ascontiguousarray(b.T)), N, dev(H, np.ascontiguousarray(bl.T)), N
    nblk = (N + 63) // 64
    arr = torch.full((nblk * ((K + 63) // 64) * 4096,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    arr2 = torch.full((nblk * ((K2 + 63) // 64) * 4096,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_gemm_arrange(stream(), Bm, ldb, N, K, layout, arr)
    B.rp_op_gemm_arrange(stream(), B2m, ldb2, N, K2, layout, arr2)
    A, A2, R = dev(H, a), dev(H, u), dev(H, res)
    outs = []
    for tile, b1, b2, l1, l2 in ((1, Bm, B2m, ldb, ldb2), (6, arr, arr2, 0, 0)):
        Cm = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 0, A, b1, Cm, M, N, K, K, l1, N, A2=A2, B2=b2, K2=K2, lda2=K2, ldb2=l2, R=R, ldr=N, tile=tile)
        C32 = torch.full((M, N), 0.5, dtype=torch.float32, device="cuda:0")
        B.rp_op_gemm(stream(), layout, 1, A, b1, C32, M, N, K, K, l1, N, alpha=0.25, beta=1, A2=A2, B2=b2, K2=K2, lda2=K2, ldb2=l2, tile=tile)
        Cp = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")     # no second pair
        B.rp_op_gemm(stream(), layout, 0, A, b1, Cp, M, N, K, K, l1, N, tile=tile)
        torch.cuda.synchronize()
        outs.append((H.to_f32(Cm), C32.cpu().numpy(), H.to_f32(Cp)))
    assert rel_l2(outs[1][0], ref + res) < 4e-3
    assert rel_l2(outs[1][1], 0.25 * ref + 0.5) < 1e-5
    assert rel_l2(outs[1][2], a.astype(np.float64) @ b.T.astype(np.float64)) < 4e-3
    for got, want in zip(outs[1], outs[0]):
        np.testing.assert_array_equal(got, want)
    # the arrangement itself: zero padding and element order, from the definition
    arr_h = H.to_f32(arr).reshape(nblk, (K + 63) // 64, 4, 2, 64, 8)
    want = np.zeros((nblk * 64, ((K + 63) // 64) * 64), dtype=np.float32)
    want[:N, :K] = b
    want = want.reshape(nblk, 2, 32, (K + 63) // 64, 4, 2, 8)          # blk, j, lr, kt, ks, lk, e
    want = want.transpose(0, 3, 4, 1, 5, 2, 6).reshape(nblk, (K + 63) // 64, 4, 2, 64, 8)   # lane = lk * 32 + lr
    np.testing.assert_array_equal(arr_h, want)


def test_gemm_second_pair_residual_and_atomic(rp):
    B, H = rp
    rng = np.random.default_rng(7)
    M, N, K, K2 = 520, 392, 328, 24
    x, w = rnd(rng, (M, K)), rnd(rng, (N, K), 0.05)
    u, bl = rnd(rng, (M, K2)), rnd(rng, (N, K2), 0.1)
    res = rnd(rng, (M, N))
    ref = x.astype(np.float64) @ w.T.astype(np.float64) + u.astype(np.float64) @ bl.T.astype(np.float64) + res
    for tile in (0, 1, 5):
        Cm = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda:0")
        B.rp_op_gemm(stream(), 0, 0, dev(H, x), dev(H, w), Cm, M, N, K, K, K, N, A2=dev(H, u), B2=dev(H, bl), K2=K2,
                     lda2=K2, ldb2=K2, R=dev(H, res), ldr=N, tile=tile)
        torch.cuda.synchronize()
        assert rel_l2(H.to_f32(Cm), ref) < 4e-3, tile
    # the same with a scale on the product (the residual is not scaled)
    Cm = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_gemm(stream(), 0, 0, dev(H, x), dev(H, w), Cm, M, N, K, K, K, N, alpha=0.5, A2=dev(H, u), B2=dev(H, bl), K2=K2,
                 lda2=K2, ldb2=K2, R=dev(H, res), ldr=N, tile=1)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(Cm), 0.5 * (ref - res) + res) < 4e-3
    # NN with a second pair (activation gradient of a LoRA linear): dx = dy W + ud A
    dy, ud, a_l = rnd(rng, (M, N)), rnd(rng, (M, K2)), rnd(rng, (K2, K), 0.1)
    ref2 = dy.astype(np.float64) @ w.astype(np.float64) + ud.astype(np.float64) @ a_l.astype(np.float64)
    C2 = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_gemm(stream(), 1, 0, dev(H, dy), dev(H, w), C2, M, K, N, N, K, K, A2=dev(H, ud), B2=dev(H, a_l), K2=K2,
                 lda2=K2, ldb2=K, tile=5)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(C2), ref2) < 4e-3
    # atomic accumulation, skinny output (LoRA gradient shape): dB[N, r] += dy^T u
    C3 = torch.ones((N, K2), dtype=torch.float32, device="cuda:0")
    B.rp_op_gemm(stream(), 2, 2, dev(H, dy), dev(H, u), C3, N, K2, M, N, K2, K2)
    torch.cuda.synchronize()
    assert rel_l2(C3.cpu().numpy(), dy.T.astype(np.float64) @ u.astype(np.float64) + 1.0) < 1e-5


def test_gemm_reduction_split_merges_in_a_fixed_order(rp):
    """Weight-gradient shapes whose 256x256 tiles would leave most of the chip idle are cut along the reduction; the
    slices' partial products go through scratch memory and are added in slice order, so two runs agree bit for bit
    (Sec. 4.1.1: gradients accumulate in place over micro-batches).  Ragged M and N, K long enough for 8 slices, the
    skinny LoRA shapes with a bf16 result, and a scratch buffer too small for any split."""
    B, H = rp
    rng = np.random.default_rng(17)
    ws = torch.empty(16 << 20, dtype=torch.uint8, device="cuda:0")
    for (M, N, K) in ((520, 392, 8200), (48, 1032, 4104), (1032, 16, 4104)):
        a, b = rnd(rng, (K, M)), rnd(rng, (K, N))
        ref = a.T.astype(np.float64) @ b.astype(np.float64)
        A, Bm = dev(H, a), dev(H, b)
        outs = []
        for rep in range(2):
            ws.fill_(0xFF)                                  # NaN patterns: every partial that is read was written first
            C32 = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda:0")
            B.rp_op_gemm(stream(), 2, 1, A, Bm, C32, M, N, K, M, N, N, alpha=0.5, beta=1, split_ws=ws)
            torch.cuda.synchronize()
            outs.append(C32.clone())
        assert torch.equal(outs[0], outs[1])
        assert rel_l2(outs[0].cpu().numpy(), 0.5 * ref + 2.0) < 1e-5
        # without scratch nothing is split: same product, one pass
        C1 = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda:0")
        B.rp_op_gemm(stream(), 2, 1, A, Bm, C1, M, N, K, M, N, N, alpha=0.5, beta=1)
        torch.cuda.synchronize()
        assert rel_l2(C1.cpu().numpy(), 0.5 * ref + 2.0) < 1e-5
        # a scratch buffer that holds one slice only: no split either
        small = torch.empty(M * N * 4, dtype=torch.uint8, device="cuda:0")
        C2 = torch.full((M, N), 2.0, dtype=torch.float32, device="cuda:0")
        B.rp_op_gemm(stream(), 2, 1, A, Bm, C2, M, N, K, M, N, N, alpha=0.5, beta=1, split_ws=small)
        torch.cuda.synchronize()
        assert rel_l2(C2.cpu().numpy(), 0.5 * ref + 2.0) < 1e-5
    # skinny product with a bf16 result (LoRA down-projection: [T, h] x [3r, h]^T), NT layout
    T_, h, r3 = 2056, 1032, 48
    x, am = rnd(rng, (T_, h)), rnd(rng, (r3, h), 0.05)
    U = torch.full((T_, r3), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_gemm(stream(), 0, 3, dev(H, x), dev(H, am), U, T_, r3, h, h, h, r3, alpha=2.0, split_ws=ws)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(U), 2.0 * (x.astype(np.float64) @ am.T.astype(np.float64))) < 4e-3


def test_gemm_submatrix_views_and_tiny(rp):
    B, H = rp
    rng = np.random.default_rng(8)
    T, N, r = 72, 96, 8
    dy, u = rnd(rng, (T, N)), rnd(rng, (T, 3 * r))
    # dB_k[32, r] += dy[:, 40:72]^T u[:, r:2r]  via pointer offsets and leading dimensions
    dyt, ut = dev(H, dy), dev(H, u)
    out = torch.zeros((32, r), dtype=torch.float32, device="cuda:0")
    B.rp_op_gemm(stream(), 2, 1, dyt.data_ptr() + 40 * 2, ut.data_ptr() + r * 2, out, 32, r, T, N, 3 * r, r, beta=1)
    torch.cuda.synchronize()
    ref = dy[:, 40:72].T.astype(np.float64) @ u[:, r:2 * r].astype(np.float64)
    assert rel_l2(out.cpu().numpy(), ref) < 1e-5
    # empty problem is a no-op
    B.rp_op_gemm(stream(), 0, 0, dyt, ut, out, 0, 8, 8, 8, 8, 8)
    torch.cuda.synchronize()


# ----------------------------------------------------------------------------------------------- RMSNorm
@pytest.mark.parametrize("T,h", [(37, 256), (130, 2048), (40, 4096), (21, 5120), (1300, 512)])
def test_rmsnorm_fwd_bwd(rp, T, h):
    B, H = rp
    rng = np.random.default_rng(T + h)
    x, g, dy, dres = rnd(rng, (T, h)), synth.bf16_round(1 + 0.1 * rng.standard_normal(h).astype(np.float32)), rnd(rng, (T, h)), rnd(rng, (T, h))
    y_ref, rstd_ref = L.rmsnorm_fwd(x.astype(np.float64), g.astype(np.float64), 1e-6)
    xd, gd = dev(H, x), dev(H, g)
    y = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0")
    rstd = torch.empty(T, dtype=torch.float32, device="cuda:0")
    B.rp_op_rmsnorm_fwd(stream(), xd, gd, y, rstd, T, h, 1e-6)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(y), y_ref) < 4e-3
    assert rel_l2(rstd.cpu().numpy(), rstd_ref[:, 0]) < 1e-5
    dx_ref, dg_ref = L.rmsnorm_bwd(dy.astype(np.float64), x.astype(np.float64), g.astype(np.float64), rstd_ref)
    for f32 in (0, 1):
        dx = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0")
        dg = torch.zeros(h, dtype=torch.float32, device="cuda:0")
        dyd = torch.from_numpy(dy).cuda() if f32 else dev(H, dy)
        scratch = torch.empty(1024 * h, dtype=torch.float32, device="cuda:0")
        B.rp_op_rmsnorm_bwd(stream(), dyd, f32, xd, gd, rstd, dev(H, dres), dx, dg, scratch, T, h)
        torch.cuda.synchronize()
        assert rel_l2(H.to_f32(dx), dx_ref + dres) < 4e-3
        assert rel_l2(dg.cpu().numpy(), dg_ref) < 1e-4


# ----------------------------------------------------------------------------------------------- QK-norm + RoPE
@pytest.mark.parametrize("d,a,k,use_norm", [(128, 4, 2, 1), (64, 6, 3, 1), (128, 3, 1, 0)])
def test_qknorm_rope_fwd_bwd(rp, d, a, k, use_norm):
    B, H = rp
    rng = np.random.default_rng(d + a)
    batch, seq = 2, 52
    T, base, eps = batch * seq, 1.0e6, 1e-6
    n1 = (a + 2 * k) * d
    qkv = rnd(rng, (T, n1))
    gq = synth.bf16_round(1 + 0.1 * rng.standard_normal(d).astype(np.float32))
    gk = synth.bf16_round(1 + 0.1 * rng.standard_normal(d).astype(np.float32))
    q_raw = qkv[:, : a * d].reshape(T, a, d).astype(np.float64)
    k_raw = qkv[:, a * d: (a + k) * d].reshape(T, k, d).astype(np.float64)
    if use_norm:
        qn, rq = L.rmsnorm_fwd(q_raw, gq.astype(np.float64), eps)
        kn, rk = L.rmsnorm_fwd(k_raw, gk.astype(np.float64), eps)
    else:
        qn, kn = q_raw, k_raw
    q_ref, k_ref = L.rope_fwd(qn, batch, seq, base), L.rope_fwd(kn, batch, seq, base)

    cs = torch.empty((seq, d // 2, 2), dtype=torch.float32, device="cuda:0")
    B.rp_op_rope_table(stream(), cs, seq, d, base)
    qkvd = dev(H, qkv)
    qo = torch.empty((T, a * d), dtype=torch.bfloat16, device="cuda:0")
    ko = torch.empty((T, k * d), dtype=torch.bfloat16, device="cuda:0")
    rstd_q = torch.zeros((T, a), dtype=torch.float32, device="cuda:0")
    rstd_k = torch.zeros((T, k), dtype=torch.float32, device="cuda:0")
    gqd, gkd = dev(H, gq), dev(H, gk)
    B.rp_op_qknorm_rope(stream(), 0, d, qkvd, qkvd.data_ptr() + a * d * 2, n1, n1, qo, ko, a * d, k * d, gqd, gkd, rstd_q,
                        rstd_k, None, None, 0, None, None, None, cs, T, seq, a, k, use_norm, eps)
    torch.cuda.synchronize()
    cs_ref_c, cs_ref_s = L.rope_angles(seq, d, base, np.float64)
    assert np.max(np.abs(cs.cpu().numpy()[..., 0] - cs_ref_c)) < 2e-7
    assert np.max(np.abs(cs.cpu().numpy()[..., 1] - cs_ref_s)) < 2e-7
    assert rel_l2(H.to_f32(qo).reshape(T, a, d), q_ref) < 4e-3
    assert rel_l2(H.to_f32(ko).reshape(T, k, d), k_ref) < 4e-3

    # backward: gradients of the rotated heads -> gradients of the raw heads (written into a fused [T, n1] buffer)
    dq_r, dk_r = rnd(rng, (T, a, d)), rnd(rng, (T, k, d))
    dqn = L.rope_bwd(dq_r.astype(np.float64), batch, seq, base)
    dkn = L.rope_bwd(dk_r.astype(np.float64), batch, seq, base)
    if use_norm:
        dq_ref, dgq_ref = L.rmsnorm_bwd(dqn, q_raw, gq.astype(np.float64), rq)
        dk_ref, dgk_ref = L.rmsnorm_bwd(dkn, k_raw, gk.astype(np.float64), rk)
    else:
        dq_ref, dk_ref = dqn, dkn
    dqkv = torch.zeros((T, n1), dtype=torch.bfloat16, device="cuda:0")
    dgq = torch.zeros(d, dtype=torch.float32, device="cuda:0")
    dgk = torch.zeros(d, dtype=torch.float32, device="cuda:0")
    B.rp_op_qknorm_rope(stream(), 1, d, dev(H, dq_r.reshape(T, -1)), dev(H, dk_r.reshape(T, -1)), a * d, k * d, dqkv,
                        dqkv.data_ptr() + a * d * 2, n1, n1, gqd, gkd, rstd_q, rstd_k, qkvd, qkvd.data_ptr() + a * d * 2, n1,
                        dgq, dgk, torch.empty(1024 * 2 * d, dtype=torch.float32, device="cuda:0"), cs, T, seq, a, k, use_norm, eps)
    torch.cuda.synchronize()
    out = H.to_f32(dqkv)
    assert rel_l2(out[:, : a * d].reshape(T, a, d), dq_ref) < 4e-3
    assert rel_l2(out[:, a * d: (a + k) * d].reshape(T, k, d), dk_ref) < 4e-3
    assert np.all(out[:, (a + k) * d:] == 0)
    if use_norm:
        assert rel_l2(dgq.cpu().numpy(), dgq_ref) < 1e-4
        assert rel_l2(dgk.cpu().numpy(), dgk_ref) < 1e-4


# ----------------------------------------------------------------------------------------------- SwiGLU
def test_swiglu_fwd_bwd(rp):
    B, H = rp
    rng = np.random.default_rng(5)
    T, m = 75, 688
    gu, dact = rnd(rng, (T, 2 * m), 2.0), rnd(rng, (T, m))
    g64, u64 = gu[:, :m].astype(np.float64), gu[:, m:].astype(np.float64)
    gud = dev(H, gu)
    act = torch.empty((T, m), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_swiglu_fwd(stream(), gud, act, T, m)
    dgu = torch.empty((T, 2 * m), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_swiglu_bwd(stream(), dev(H, dact), gud, dgu, T, m)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(act), L.swiglu_fwd(g64, u64)) < 4e-3
    dg_ref, du_ref = L.swiglu_bwd(dact.astype(np.float64), g64, u64)
    assert rel_l2(H.to_f32(dgu), np.concatenate([dg_ref, du_ref], axis=1)) < 4e-3


# ----------------------------------------------------------------------------------------------- attention
# the last two cases are long sequences (8192 tokens and more): many key tiles per query tile, fold order of the grid
@pytest.mark.parametrize("d,a,kh,batch,seq", [(128, 4, 2, 1, 328), (64, 4, 2, 2, 136), (128, 8, 1, 1, 200), (128, 2, 2, 1, 8),
                                              (128, 2, 1, 1, 8264), (64, 1, 1, 1, 8192)])
def test_attention_fwd_bwd(rp, d, a, kh, batch, seq):
    B, H = rp
    rng = np.random.default_rng(d + a + seq)
    T = batch * seq
    q, k, v = rnd(rng, (T, a, d)), rnd(rng, (T, kh, d)), rnd(rng, (T, kh, d))
    do = rnd(rng, (T, a, d))
    q64, k64, v64 = q.astype(np.float64), k.astype(np.float64), v.astype(np.float64)
    o_ref, P, lse_ref = L.attention_fwd(q64, k64, v64, batch, seq)
    dq_ref, dk_ref, dv_ref = L.attention_bwd(do.astype(np.float64), q64, k64, v64, o_ref, P, batch, seq)
    # k and v live side by side in one buffer (row stride 2*kh*d), as in the fused projection output
    kv = np.concatenate([k.reshape(T, -1), v.reshape(T, -1)], axis=1)
    qd_, kvd = dev(H, q.reshape(T, -1)), dev(H, kv)
    kp, vp, ldkv = kvd.data_ptr(), kvd.data_ptr() + kh * d * 2, 2 * kh * d
    o = torch.zeros((T, a * d), dtype=torch.bfloat16, device="cuda:0")
    lse = torch.zeros((batch, a, seq), dtype=torch.float32, device="cuda:0")
    B.rp_op_attn_fwd(stream(), qd_, kp, vp, o, lse, a * d, ldkv, ldkv, a * d, batch, seq, a, kh, d)
    torch.cuda.synchronize()
    assert rel_l2(H.to_f32(o).reshape(T, a, d), o_ref) < 6e-3
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) < 2e-3
    dq = torch.zeros((T, a * d), dtype=torch.bfloat16, device="cuda:0")
    dkv = torch.zeros((T, 2 * kh * d), dtype=torch.bfloat16, device="cuda:0")
    delta = torch.zeros((batch, a, seq), dtype=torch.float32, device="cuda:0")
    scratch = torch.full((2, T, a * d), float("nan"), dtype=torch.float32, device="cuda:0") if a != kh else None
    B.rp_op_attn_bwd(stream(), qd_, kp, vp, o, dev(H, do.reshape(T, -1)), lse, delta, dq, dkv, dkv.data_ptr() + kh * d * 2,
                     scratch, a * d, ldkv, ldkv, a * d, a * d, a * d, ldkv, ldkv, batch, seq, a, kh, d)
    torch.cuda.synchronize()
    dkv_h = H.to_f32(dkv)
    assert rel_l2(H.to_f32(dq).reshape(T, a, d), dq_ref) < 1e-2
    assert rel_l2(dkv_h[:, : kh * d].reshape(T, kh, d), dk_ref) < 1e-2
    assert rel_l2(dkv_h[:, kh * d:].reshape(T, kh, d), dv_ref) < 1e-2


# ----------------------------------------------------------------------------------------------- MoE routing and plan
@pytest.mark.parametrize("T,E,k", [(1, 8, 2), (200, 8, 2), (1064, 128, 8), (3000, 32, 4), (77, 6, 6), (520, 1024, 3)])
def test_moe_route_and_plan_are_exact(rp, T, E, k):
    """Index work, compared bit for bit: the selected experts (with planted exact ties), the stable counting sort of
    the (token, choice) entries, the per-expert segments and the table of 256-row tiles.  The routing weights are
    floating point and compared to fp32 rounding."""
    B, H = rp
    rng = np.random.default_rng(9000 + T + E)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    if T > 3 and E >= 4:                       # exact ties: the lower expert index must win
        logits[1, :] = 0.25
        logits[2, E - 1] = logits[2, 0] = 3.0
    n = T * k
    dv = "cuda:0"
    d_logits = torch.from_numpy(logits).to(dv)
    i32 = lambda m: torch.full((max(m, 1),), -7, dtype=torch.int32, device=dv)
    idx, counts, seg, ntiles, slot_of, row_tok = i32(n), i32(E), i32(E + 1), i32(1), i32(n), i32(n)
    max_tiles = n // 256 + E + 1
    tab = torch.full((max_tiles, 4), -7, dtype=torch.int32, device=dv)
    hist = i32((n + 511) // 512 * E)
    w = torch.zeros(n, dtype=torch.float32, device=dv)
    B.rp_op_moe_route_plan(stream(), d_logits, T, E, k, idx, w, counts, seg, tab, ntiles, slot_of, row_tok, hist)
    torch.cuda.synchronize()
    ref_idx, ref_w = L.moe_route(logits.astype(np.float64), k)
    got_idx = idx.cpu().numpy()[:n].reshape(T, k)
    assert np.array_equal(got_idx, ref_idx)
    assert np.max(np.abs(w.cpu().numpy()[:n].reshape(T, k) - ref_w)) < 1e-6
    flat = ref_idx.reshape(-1)
    ref_counts = np.bincount(flat, minlength=E)
    ref_seg = np.concatenate([[0], np.cumsum(ref_counts)])
    order = np.argsort(flat, kind="stable")           # slot -> entry
    ref_slot = np.empty(n, dtype=np.int64)
    ref_slot[order] = np.arange(n)
    assert np.array_equal(counts.cpu().numpy(), ref_counts)
    assert np.array_equal(seg.cpu().numpy(), ref_seg)
    assert np.array_equal(slot_of.cpu().numpy()[:n], ref_slot)
    assert np.array_equal(row_tok.cpu().numpy()[:n], order // k)
    tiles = []
    for e in range(E):
        for r0 in range(0, int(ref_counts[e]), 256):
            tiles.append((e, int(ref_seg[e]) + r0, min(256, int(ref_counts[e]) - r0), 0))
    assert int(ntiles.item()) == len(tiles) <= max_tiles
    assert np.array_equal(tab.cpu().numpy()[:len(tiles)], np.array(tiles, dtype=np.int32).reshape(-1, 4))
