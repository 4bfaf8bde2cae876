"""Grouped products on either side of the line up to which the experts' weights are read non-temporally: 112 rows per entry of the
tile table (rows / 256 + experts + 1 entries).  Eight experts, two per token, widths that are no multiples of the tiles or of the K
tile, so that experts with one tile and experts with two occur on both sides; against the oracle, bound 2e-2 as for every stage."""
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

E, K = 8, 2


@pytest.fixture(scope="module")
def hz():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import harness
    return harness


@pytest.mark.parametrize("tokens, once", [(8, True), (896, True), (904, False), (1280, False)])
def test_moe_stage_at_the_line(hz, tokens, once):
    rows = tokens * K
    assert (rows <= 112 * (rows // 256 + E + 1)) == once
    c = dict(n_layers=1, hidden=360, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=360, vocab=0, n_experts=E, top_k=K, lora_rank=0,
             lora=(), train_base=0, batch=1, seq=tokens, x_from="normal")
    wl = synth.make_workload(c, 2100 + tokens, gains_random=True)
    errs = pu.compare_chain(pu.oracle_chain(c, wl), pu.gpu_chain(c, wl, hz), c)
    assert len(errs) == 3, sorted(errs)
