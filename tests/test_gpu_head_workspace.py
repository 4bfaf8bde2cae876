"""A frozen LM head keeps the probabilities of the whole vocabulary when its workspace holds them, and one chunk's in a workspace too
small for that: the same results up to the order of fp32 sums."""
import numpy as np
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("one_chunk", [False, True])
def test_flags_are_used_again_with_and_without_kept_probabilities(one_chunk):
    """66 chunks of 256 rows and a ragged one, a reference that moves in chunk 1 and, behind the same flag, in chunk 65: the sums formed so
    far (one chunk's probabilities in the workspace) or all probabilities are rescaled.  The input is +-1 with unit gains, which bf16
    holds, because logits of several hundred turn its rounding into factors; bound 2e-2 as for the other heads."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness
    seq, vocab = 72, 66 * 256 + 40
    c = dict(n_layers=0, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=256, vocab=vocab, n_experts=0, top_k=0, lora_rank=0,
             lora=(), train_base=0, batch=1, seq=seq, x_from="normal", head_chunk=256)
    wl = synth.make_workload(c, 85, gains_random=True)
    wl["x"] = np.where(wl["x"] < 0, np.float32(-1), np.float32(1))
    wl["head"]["gf"] = np.ones_like(wl["head"]["gf"])
    W = wl["head"]["Wv"]
    W[256:512] *= 100.0
    W[65 * 256:66 * 256] *= 250.0
    wl["head"]["Wv"] = synth.bf16_round(W)
    wl["labels"][1::9], wl["labels"][2::9], wl["labels"][::7] = 65 * 256 + 3, 300, -100
    ref = pu.oracle_chain(c, wl)
    cfg = harness.cfg_from_dict(c, with_head=True)
    r = harness.StageRunner(cfg, 1, seq)
    try:
        r.upload(r.pinned_blob(wl["layers"], wl["head"]))
        x, labels = harness.bf16_tensor(wl["x"], r.device), torch.from_numpy(wl["labels"]).to(r.device)
        nbytes = B.rp_query_least_workspace(cfg, 1, seq)[2] if one_chunk else r.wsbytes
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=r.device)      # NaN wherever nothing was written
        loss, dx = torch.zeros(1, device=r.device), torch.empty_like(x)
        torch.cuda.synchronize()
        B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, x, labels, loss, dx, None, 1.0, 1, seq, ws, nbytes)
        r.sync()
        loss, dx = float(loss.item()), harness.to_f32(dx)
    finally:
        r.close()
    assert abs(loss - ref["loss"]) <= 1e-4 * abs(ref["loss"])
    assert np.linalg.norm(dx - ref["head_dx"]) <= 2e-2 * np.linalg.norm(ref["head_dx"])


@pytest.mark.parametrize("seq,vocab", [(72, 9 * 256 + 40), (520, 4096), (8, 264)])
def test_frozen_head_in_a_workspace_for_one_chunk(seq, vocab):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness
    c = dict(n_layers=0, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=256, vocab=vocab, n_experts=0, top_k=0, lora_rank=0,
             lora=(), train_base=0, batch=1, seq=seq, x_from="normal", head_chunk=256)
    wl = synth.make_workload(c, 91, gains_random=True)
    wl["labels"][::5] = -100
    ref = pu.oracle_chain(c, wl, grad_scale=8.0)
    cfg = harness.cfg_from_dict(c, with_head=True)
    r = harness.StageRunner(cfg, 1, seq)
    try:
        r.upload(r.pinned_blob(wl["layers"], wl["head"]))
        x, labels = harness.bf16_tensor(wl["x"], r.device), torch.from_numpy(wl["labels"]).to(r.device)
        up = lambda n: (n + 255) // 256 * 256  # noqa: E731
        small = r.wsbytes - up(vocab * seq * 2) + up(256 * seq * 2)
        got = []
        for ws in (r.wsbytes, small):
            loss, dx = torch.zeros(1, device=r.device), torch.empty_like(x)
            torch.cuda.synchronize()
            B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, x, labels, loss, dx, None, 8.0, 1, seq, r.ws, ws)
            r.sync()
            got.append((float(loss.item()), harness.to_f32(dx)))
        with pytest.raises(RuntimeError):
            B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, x, labels, loss, dx, None, 8.0, 1, seq, r.ws, small - 256)
    finally:
        r.close()
    norm = np.linalg.norm(ref["head_dx"])
    for loss, dx in got:
        assert abs(loss - ref["loss"]) <= 1e-4 * abs(ref["loss"])
        assert np.linalg.norm(dx - ref["head_dx"]) <= 2e-2 * norm
    assert got[0][0] == got[1][0]                                        # the loss comes from the same logits
    # the sums are fp32 in another order; what is left is a bf16 rounding that falls the other way on few elements (2^-9 of them each)
    assert np.linalg.norm(got[0][1] - got[1][1]) <= 2e-3 * norm
