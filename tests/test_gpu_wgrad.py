"""Weight gradients of a layer in one launch against one launch each (a workspace without the optional regions): the same fp32 sums of
the same bf16 products, in another order."""
import re

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("layers,batch,seq,h,a,kh,d,ffn,r", [
    (1, 1, 520, 1288, 20, 4, 64, 3080, 0),     # tiles ragged in both directions, a reduction that ends inside a K tile
    (2, 2, 300, 1024, 8, 8, 128, 2048, 0),     # no groups; the second layer's gradients come first
    (2, 1, 1000, 768, 12, 2, 64, 4096, 8),     # adapters on q and down beside the base weights
])
def test_weight_gradients_in_one_launch(layers, batch, seq, h, a, kh, d, ffn, r):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T = batch * seq
    cfg = B.make_cfg(layers, h, a, kh, d, ffn, lora_rank=r, lora=("q", "down") if r else ())
    s = H.StageRunner(cfg, batch, seq)
    g = torch.Generator(device="cuda:0").manual_seed(h)
    s.slots[0].view(torch.bfloat16).normal_(0.0, 0.04, generator=g)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)
    dy = torch.empty_like(x).normal_(0.0, 1.0, generator=g)
    torch.cuda.synchronize()
    s.bind()
    with pytest.raises(B.RpError) as e:
        B.rp_stage_backward(s.ctx, 0, B.PHASE_BOTH, x, dy, torch.empty_like(x), None, s.grads, None, None, batch, seq, s.ws, 256)
    need = int(re.search(r"< (\d+)", str(e.value)).group(1))
    ds = 0
    if d == 128:                                                       # leave dS out: it rounds dQ differently
        n = (seq + 127) // 128
        ds = n * (n + 1) * 16384 * a * batch
    out = []
    for nbytes in (need, s.wsbytes - ds, s.wsbytes - ds):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda:0")
        dx, gr = torch.full_like(x, float("nan")), torch.full_like(s.grads, 0.5)
        torch.cuda.synchronize()
        B.rp_trace_start(s.ctx, 512)
        B.rp_stage_backward(s.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, gr, None, None, batch, seq, ws, nbytes)
        rec = B.rp_trace_stop(s.ctx, 512)
        out.append((dx, gr, len(rec)))
    s.close()
    assert out[1][2] < out[0][2]                                       # fewer launches recorded
    assert torch.equal(out[1][0], out[2][0]) and torch.equal(out[1][1], out[2][1])
    assert torch.equal(out[0][0], out[1][0])
    a0, a1 = out[0][1].double() - 0.5, out[1][1].double() - 0.5
    assert float((a1 - a0).norm() / a0.norm()) < 1e-5
    # tensor by tensor
    for layer in range(layers):
        for name in ("WQKV", "WO", "WGU", "WD", "G1", "G2", "GQ", "GK") + (("LA_Q", "LB_Q", "LA_DOWN", "LB_DOWN") if r else ()):
            off, n = B.rp_grad_layout(cfg, layer, B.T[name])
            b0, b1 = a0[off // 4:off // 4 + n], a1[off // 4:off // 4 + n]
            assert float((b1 - b0).norm() / b0.norm()) < 1e-5, name


@pytest.mark.parametrize("names", [("q", "k", "v", "o", "gate", "up", "down"), ("o",), ("down", "v"), ("gate",)])
@pytest.mark.parametrize("batch,seq,frozen", [(1, 72, 1), (2, 300, 0), (1, 4104, 1)])      # 4104: dA does not wait any more
def test_adapter_gradients_that_wait_for_the_next_projection(names, batch, seq, frozen):
    """An adapter's dA joins the next projection's first launch, whose dU then goes to the other of two buffers; at the least workspace it
    has a launch of its own.  Tensor by tensor and layer by layer, also where the next projections have no adapter.  Sums of small products
    are cut elsewhere, and a bf16 rounding that falls the other way carries on: at most every rounding behind it is another one, seven
    in a layer (dgu, dn, dy, dout, dq, dqkv, dU), 1.1e-3 each in the mean square, on both sides, over three layers: sqrt(2 * 7 * 3) * 1.1e-3 =
    7e-3, bound 8e-3.  (Measured 2e-3; a dA of the wrong dU is off by its whole norm.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h, layers = batch * seq, 512, 3
    cfg = B.make_cfg(layers, h, 8, 2, 64, 1024, lora_rank=16, lora=names, train_base=1 - frozen)
    s = H.StageRunner(cfg, batch, seq)
    g = torch.Generator(device="cuda:0").manual_seed(seq + len(names))
    s.slots[0].view(torch.bfloat16).normal_(0.0, 0.04, generator=g)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)
    dy = torch.empty_like(x).normal_(0.0, 1.0, generator=g)
    torch.cuda.synchronize()
    s.bind()
    out = []
    for nbytes in (B.rp_query_least_workspace(cfg, batch, seq)[1], s.wsbytes):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda:0")
        dx, gr = torch.full_like(x, float("nan")), torch.zeros_like(s.grads)
        torch.cuda.synchronize()
        B.rp_stage_backward(s.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, gr, None, None, batch, seq, ws, nbytes)
        s.sync()
        out.append((dx.double(), gr.double()))
    s.close()
    assert float((out[1][0] - out[0][0]).norm() / out[0][0].norm()) < 8e-3
    for layer in range(layers):
        for n in names:
            for t in ("LA_", "LB_"):
                off, cnt = B.rp_grad_layout(cfg, layer, B.T[t + n.upper()])
                a0, a1 = out[0][1][off // 4:off // 4 + cnt], out[1][1][off // 4:off // 4 + cnt]
                assert float((a1 - a0).norm() / a0.norm()) < 8e-3, (layer, t + n)


def test_rows_too_far_apart_for_the_shared_launch():
    """The shared launch addresses the 256 rows of an output tile with 31-bit offsets.  Rows of 2097280 fp32 numbers (the output projection of 16385
    heads, whose last tile is ragged) are further apart than that: such a gradient is computed by itself, with the sums of the least workspace."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h = 8, 256
    cfg = B.make_cfg(1, h, 16385, 5, 128, 512, lora_rank=0, lora=())
    s = H.StageRunner(cfg, 1, T)
    g = torch.Generator(device="cuda:0").manual_seed(1)
    s.slots[0].view(torch.bfloat16).normal_(0.0, 0.04, generator=g)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)
    dy = torch.empty_like(x).normal_(0.0, 1.0, generator=g)
    torch.cuda.synchronize()
    s.bind()
    off, n = B.rp_grad_layout(cfg, 0, B.T["WO"])
    out = []
    for nbytes in (B.rp_query_least_workspace(cfg, 1, T)[1], s.wsbytes):
        s.grads.fill_(0.5)
        torch.cuda.synchronize()
        B.rp_trace_start(s.ctx, 512)
        B.rp_stage_backward(s.ctx, 0, B.PHASE_BOTH, x, dy, torch.empty_like(x), None, s.grads, None, None, 1, T, s.ws, nbytes)
        assert not any(t[0] == "gemm_wgrad_TN" for t in B.rp_trace_stop(s.ctx, 512))
        out.append(s.grads[off // 4:off // 4 + n].view(h, n // h) - 0.5)
    s.close()
    # the last heads' columns by themselves: the whole gradient would hide one wrong tile
    for part in (slice(0, None), slice(n // h - 128, None), slice(2064384, 2064640)):
        a, b = out[0][:, part], out[1][:, part]
        assert float(a.norm()) > 0 and float((b - a).norm() / a.norm()) < 1e-5
    rows = out[1][-1], out[0][-1]
    assert float((rows[0] - rows[1]).norm() / rows[1].norm()) < 1e-5
