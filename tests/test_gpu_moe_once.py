"""Grouped products on either side of the lines up to which the experts' weights are loaded non-temporally: 240 rows per expert on
average, and more than 200 MiB of expert weights in the stage.  Which kernel ran is read from the timeline.  Widths that are no multiples
of the tiles or of the K tile, experts with one tile and with two on both sides; against the oracle, bound 2e-2 as for every stage."""
import pytest

import parity_util as pu
import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def hz():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import harness
    return harness


def _names(hz, c, T):
    from paper_2604_27085_amd import binding as B
    r = hz.StageRunner(hz.cfg_from_dict(c), c["batch"], c["seq"])
    try:
        r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
        x = torch.empty((T, c["hidden"]), dtype=torch.bfloat16, device=r.device).normal_()
        dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
        router = torch.randn((c["n_layers"], T, c["n_experts"]), device=r.device)
        torch.cuda.synchronize()
        r.bind()
        B.rp_trace_start(r.ctx, 512)
        B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, None, router, None, c["batch"], c["seq"], r.ws, r.wsbytes)
        return [t[0] for t in B.rp_trace_stop(r.ctx, 512)]
    finally:
        r.close()


def _cfg(layers, E, K, width, tokens):
    return dict(n_layers=layers, hidden=width, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=width, vocab=0, n_experts=E, top_k=K, lora_rank=0,
                lora=(), train_base=0, batch=1, seq=tokens, x_from="normal")


# 6 E h m bytes per layer: 8 experts of 2088 are 199.6 MiB, of 2096 201.1 MiB; two layers of 1480 are 200.5 MiB
@pytest.mark.parametrize("layers,E,width,tokens,once", [
    (1, 8, 2096, 960, True), (1, 8, 2096, 968, False),     # 240 rows per expert, and two more
    (1, 8, 2088, 8, False), (1, 8, 2096, 8, True),         # the weights
    (2, 8, 1480, 64, True), (1, 8, 1480, 64, False),
])
def test_where_the_lines_lie(hz, layers, E, width, tokens, once):
    names = _names(hz, _cfg(layers, E, 2, width, tokens), tokens)
    ran = [n for n in names if n.startswith("gemm_grouped") and n != "gemm_grouped_pair"]
    assert ran and all(("once" in n) == once for n in ran), ran


@pytest.mark.parametrize("E,width,tokens,once", [
    (8, 360, 8, False), (8, 360, 896, False), (8, 360, 904, False), (8, 360, 1280, False),
    (72, 712, 8, True), (72, 712, 1000, True),
])
def test_moe_stage_at_the_line(hz, E, width, tokens, once):
    c = _cfg(1, E, 2, width, tokens)
    assert (tokens * 2 <= 240 * E and 6 * E * width * width > 200 * 2 ** 20) == once
    wl = synth.make_workload(c, 2100 + tokens, gains_random=True)
    errs = pu.compare_chain(pu.oracle_chain(c, wl), pu.gpu_chain(c, wl, hz), c)
    assert len(errs) == 3, sorted(errs)
