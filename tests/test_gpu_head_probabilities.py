"""The LM head's probabilities straight from the four-wave kernel's registers (reductions of 2048 take it for any number of tiles): vocabulary
chunks that end inside a 128-row block and before one, tokens that end inside a 16-column tile and inside a 128-column block, labels in
every 16-row tile, in the last row and in none."""
import numpy as np
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("seq,vocab", [(72, 256 + 200), (264, 512), (392, 256 + 72)])
def test_probabilities_from_registers(seq, vocab):
    """Bounds as for the other heads: 1e-4 on the loss (fp32 sums), 2e-2 on bf16 results."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness
    c = dict(n_layers=0, hidden=2048, n_q_heads=16, n_kv_heads=8, head_dim=128, ffn=256, vocab=vocab, n_experts=0, top_k=0, lora_rank=0,
             lora=(), train_base=0, batch=1, seq=seq, x_from="normal", head_chunk=256)
    wl = synth.make_workload(c, 93, gains_random=True)
    wl["labels"][:] = (np.arange(seq) * 37 + 5) % vocab
    wl["labels"][::11], wl["labels"][1::13] = -100, vocab - 1
    assert len(set(wl["labels"] // 16)) > vocab // 20
    ref = pu.oracle_chain(c, wl, grad_scale=8.0)
    cfg = harness.cfg_from_dict(c, with_head=True)
    r = harness.StageRunner(cfg, 1, seq)
    try:
        r.upload(r.pinned_blob(wl["layers"], wl["head"]))
        x, labels = harness.bf16_tensor(wl["x"], r.device), torch.from_numpy(wl["labels"]).to(r.device)
        ws = torch.full((r.wsbytes,), 255, dtype=torch.uint8, device=r.device)      # NaN wherever nothing was written
        loss, dx = torch.zeros(1, device=r.device), torch.empty_like(x)
        torch.cuda.synchronize()
        B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, x, labels, loss, dx, None, 8.0, 1, seq, ws, r.wsbytes)
        r.sync()
        loss, dx = float(loss.item()), harness.to_f32(dx)
    finally:
        r.close()
    assert abs(loss - ref["loss"]) <= 1e-4 * abs(ref["loss"])
    assert np.linalg.norm(dx - ref["head_dx"]) <= 2e-2 * np.linalg.norm(ref["head_dx"])
