"""The per-kernel timeline of a stage call: what it records is what was launched, with the bytes that the launch moves."""
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (batch, seq, query heads, kv heads, head dimension) -> partials per token that the dK/dV workgroups leave (0: none)
@pytest.mark.parametrize("batch,seq,a,kh,d,partials", [
    (32, 300, 16, 4, 128, 0),     # a workgroup takes a whole group of four
    (16, 300, 64, 8, 64, 32),     # two heads of eight
    (24, 300, 64, 8, 64, 16),     # four heads of eight
    (1, 264, 8, 2, 128, 8),       # one head
    (1, 264, 4, 4, 128, 0),       # no groups
    (1, 128, 4, 2, 64, 0),        # groups of two in one key tile
    (4, 256, 16, 8, 128, 0),      # in two, 64 heads in all
    (3, 256, 20, 10, 64, 20),     # 60 heads
    (3, 160, 16, 8, 128, 0),      # 48 heads, enough at head dimension 128
    (1, 256, 4, 2, 128, 4),
])
def test_reduction_of_dkv_partials_is_recorded_as_launched(batch, seq, a, kh, d, partials):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    c = synth.shrink(synth.CONFIGS["C1"], n_layers=1, hidden=256, ffn=256, n_q_heads=a, n_kv_heads=kh, head_dim=d, vocab=0, seq=seq, batch=batch)
    r = H.StageRunner(H.cfg_from_dict(c), batch, seq)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((batch * seq, 256), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
    torch.cuda.synchronize()
    r.bind()
    B.rp_trace_start(r.ctx, 256)
    B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, r.grads, None, None, batch, seq, r.ws, r.wsbytes)
    rec = [t for t in B.rp_trace_stop(r.ctx, 256) if t[0] == "attn_dkv_reduce"]
    r.close()
    # fp32 partials of dk and dv read, bf16 sums written
    want = [batch * seq * (2 * 4.0 * partials * d + 2 * 2.0 * kh * d)] if partials else []
    assert [t[2] for t in rec] == want


# A layer's large weight gradients share a launch where the tile model finds that cheaper; one that is alone never does.
@pytest.mark.parametrize("h,m,T,joined", [(2048, 6144, 512, True), (256, 1536, 264, False)])
def test_weight_gradients_are_recorded_as_launched(h, m, T, joined):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    c = synth.shrink(synth.CONFIGS["C1"], n_layers=1, hidden=h, ffn=m, n_q_heads=4, n_kv_heads=2, head_dim=64, vocab=0, seq=T, batch=1, lora_rank=0, lora=())
    r = H.StageRunner(H.cfg_from_dict(c), 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
    torch.cuda.synchronize()
    r.bind()
    B.rp_trace_start(r.ctx, 256)
    B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, r.grads, None, None, 1, T, r.ws, r.wsbytes)
    rec = [t for t in B.rp_trace_stop(r.ctx, 256) if t[0].endswith("_TN")]
    r.close()
    if joined:      # those of gate and up, down, and whatever else is large; the others share a launch with other small products
        assert [t[0] for t in rec] == ["gemm_wgrad_TN"]
        assert rec[0][1] >= 2.0 * T * 3 * h * m
    else:           # gate and up alone, on the tile that the product picks by itself
        assert len(rec) == 1 and rec[0][0] not in ("gemm_wgrad_TN", "gemm_256x256_TN")
        assert rec[0][1] == 2.0 * T * 2 * h * m and rec[0][2] == 2.0 * T * (2 * m + h) + 8.0 * 2 * m * h


@pytest.mark.parametrize("m,joined", [(4096, True), (4104, False)])
def test_an_adapter_gradient_that_waited_and_the_next_projection(m, joined):
    """An adapter on down only: its dA waits for the next projection, which has no small products of its own and whose dX, narrow at 64
    tokens, is drawn into a launch with it up to a weight of 16 MiB, and is left alone above."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h = 64, 1024
    r = H.StageRunner(B.make_cfg(1, h, 8, 2, 128, m, lora_rank=16, lora=("down",), train_base=0), 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
    torch.cuda.synchronize()
    r.bind()
    B.rp_trace_start(r.ctx, 256)
    B.rp_stage_backward(r.ctx, 0, B.PHASE_BACKWARD | B.PHASE_RECOMPUTE, x, dy, dx, None, r.grads, None, None, 1, T, r.ws, r.wsbytes)
    rec = B.rp_trace_stop(r.ctx, 256)
    r.close()
    wide = [t for t in rec if t[1] == 2.0 * T * 2 * m * h]      # gate and up: forward and dX
    assert sorted(t[0][-3:] for t in wide) == (["_NT"] if joined else ["_NN", "_NT"])
    assert any(t[1] > 2.0 * T * 2 * m * h for t in rec if t[0] == "gemm_group") == joined


def test_an_adapter_gradient_that_waited_joins_a_small_weight_gradient():
    """Adapters on q and v, trained weights: the second layer's dA waits for the first layer's down, whose weight gradient is small enough
    for a shared launch; the first layer's own has no projection behind it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h, m, rank = 512, 256, 688, 8
    r = H.StageRunner(B.make_cfg(2, h, 4, 2, 64, m, lora_rank=rank, lora=("q", "v"), train_base=1), 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
    torch.cuda.synchronize()
    r.bind()
    B.rp_trace_start(r.ctx, 256)
    B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, r.grads, None, None, 1, T, r.ws, r.wsbytes)
    rec = B.rp_trace_stop(r.ctx, 256)
    r.close()
    dA = 2.0 * T * 2 * rank * h
    assert sum(t[0].endswith("_TN") and t[1] == dA for t in rec) == 1
    assert any(t[0] == "gemm_group" and t[1] >= dA + 2.0 * T * h * m for t in rec)
