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
        for name in ("WQKV", "WO", "WGU", "WD", "G1", "G2", "GQ", "GK"):
            off, n = B.rp_grad_layout(cfg, layer, B.T[name])
            b0, b1 = a0[off // 4:off // 4 + n], a1[off // 4:off // 4 + n]
            assert float((b1 - b0).norm() / b0.norm()) < 1e-5, name
