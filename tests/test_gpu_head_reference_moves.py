"""A head whose reference exponents move by an amount that leaves weight on what was summed before: every kept probability, the normaliser
and (in a workspace for one chunk's probabilities) the sums already formed are rescaled.

x is 1 on the first 64 columns (every eighth token) or on the second 64; the weights of the first 2048 rows lie in the last 128 columns, so
their logits are all 0 and their probabilities 1 until the second chunk, where one row gives the former tokens 70 (which is what makes
the chunk run again) and one the others 9.  Those carry 2048 e^-9 / (2310 e^-9 + 1) = 20 % of
their weight in the first chunk: a factor e^-9 rounded to bf16 is off by 3.1e-3, the same way for every row.  The two rows are zero in the
last 128 columns, so dx there is that weight's alone: fp32 sums rounded to bf16, 2^-9 of each of 128 different values, unbiased -- 1e-4
in their scale, bound 5e-4.  Rows of the weight gradient whose logit is 0 get the same probability in both chunks, so the scale between
them is 1 up to the bf16 rounding of e^-9's neighbourhood on the side that is not rescaled, which is a power of two as well."""
import numpy as np
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _scale(got, ref):
    got, ref = np.asarray(got, np.float64).ravel(), np.asarray(ref, np.float64).ravel()
    return float(got @ ref / (ref @ ref))


# 1032 and 2056 tokens: more than one range of 1024 whose sums are added by one workgroup
@pytest.mark.parametrize("seq", [64, 1032, 2056])
@pytest.mark.parametrize("mode", ["frozen", "frozen_one_chunk", "train"])
def test_reference_moves_with_weight_on_both_sides(mode, seq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness
    train, chunk, vocab = int(mode == "train"), 2048, 2048 + 264
    c = dict(n_layers=0, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=256, vocab=vocab, n_experts=0, top_k=0, lora_rank=0,
             lora=(), train_base=train, batch=1, seq=seq, x_from="normal", head_chunk=chunk)
    wl = synth.make_workload(c, 93)
    hot = np.arange(seq) % 8 == 0
    x = np.zeros((seq, 256), np.float32)
    x[hot, :64], x[~hot, 64:128] = 1.0, 1.0
    W = wl["head"]["Wv"]
    W[:, :128] = 0.0
    W[chunk + 5, :64] = 70.0 / 128        # the normalised x is 2 there
    W[chunk + 9, 64:128] = 9.0 / 128
    W[[chunk + 5, chunk + 9], 128:] = 0.0
    wl["x"], wl["head"]["gf"] = x, np.ones(256, np.float32)
    wl["labels"][:] = chunk + 9
    ref = pu.oracle_chain(c, wl)
    cfg = harness.cfg_from_dict(c, with_head=True)
    r = harness.StageRunner(cfg, 1, seq)
    try:
        r.upload(r.pinned_blob(wl["layers"], wl["head"]))
        xt, labels = harness.bf16_tensor(x, r.device), torch.from_numpy(wl["labels"]).to(r.device)
        up = lambda n: (n + 255) // 256 * 256  # noqa: E731
        nbytes = r.wsbytes - (up(vocab * seq * 2) - up(chunk * seq * 2) if mode == "frozen_one_chunk" else 0)
        ws = torch.full((r.wsbytes,), 255, dtype=torch.uint8, device=r.device)      # NaN wherever nothing was written
        loss, dx = torch.zeros(1, device=r.device), torch.full_like(xt, float("nan"))
        torch.cuda.synchronize()
        B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, xt, labels, loss, dx, r.grads if train else None, 1.0, 1, seq, ws, nbytes)
        r.sync()
        dx, loss = harness.to_f32(dx), float(loss.item())
        gw = harness.unpack_grads(cfg, r.grads)[1]["Wv"] if train else None
    finally:
        r.close()
    assert abs(loss - ref["loss"]) <= 1e-5 * abs(ref["loss"])
    assert pu.rel_l2(dx, ref["head_dx"]) < 2e-2
    assert abs(_scale(dx[~hot, 128:], ref["head_dx"][~hot, 128:]) - 1.0) < 5e-4
    if train:
        assert pu.rel_l2(gw, ref["head_grads"]["Wv"]) < 2e-2
        rows = np.delete(gw[chunk:, 64:128], (5, 9), axis=0)
        assert abs(gw[:chunk, 64:128].mean() / rows.mean() - 1.0) < 5e-4
