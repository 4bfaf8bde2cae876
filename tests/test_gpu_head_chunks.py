"""An LM head with more vocabulary chunks than the sweep has flags (64): the flags of the first chunks are used again."""
import numpy as np
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("train_base", [0, 1])
def test_flags_are_used_again_after_64_chunks(train_base):
    """66 chunks of 256 rows and a ragged one.  The reference exponent moves in chunk 1, whose flag chunk 65 uses again, and once
    more in chunk 65; chunk 64, which has chunk 0's flag, outgrows nothing.  Logits of several hundred turn the bf16 rounding of the
    normalised input into factors of the probabilities, so the input is +-1 with unit gains, which bf16 holds.  Bounds as for the
    other heads: 2e-2 on bf16 results."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import harness
    c = dict(n_layers=0, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=256, vocab=66 * 256 + 40, n_experts=0, top_k=0, lora_rank=0,
             lora=(), train_base=train_base, batch=1, seq=72, x_from="normal", head_chunk=256)
    wl = synth.make_workload(c, 84, gains_random=True)
    wl["x"] = np.where(wl["x"] < 0, np.float32(-1), np.float32(1))
    wl["head"]["gf"] = np.ones_like(wl["head"]["gf"])
    W = wl["head"]["Wv"]
    W[256:512] *= 100.0
    W[65 * 256:66 * 256] *= 250.0
    wl["head"]["Wv"] = synth.bf16_round(W)
    wl["labels"][::7] = -100
    wl["labels"][1::9] = 65 * 256 + 3        # the chunk that uses a flag again
    wl["labels"][2::9] = 300                 # the chunk that had it first
    wl["labels"][3::9] = 66 * 256 + 39       # last row of the ragged chunk
    ref = pu.oracle_chain(c, wl, grad_scale=32.0)
    got = pu.gpu_chain(c, wl, harness, grad_scale=32.0)
    errs = pu.compare_chain(ref, got, c)
    assert {"loss", "head_dx"} <= set(errs)
    logits = wl["head"]["Wv"].astype(np.float64) @ wl["x"].astype(np.float64).T
    best = lambda lo, hi: logits[lo:hi].max(axis=0)  # noqa: E731
    assert (best(256, 512) > best(0, 256) + 60).sum() > 36 and (best(65 * 256, 66 * 256) > best(0, 65 * 256) + 60).sum() > 36
