"""Expert stages whose down projection and the gradient of its input share a launch, against the two phases run apart, where they cannot: the
same bits (of the four-wave kernel and, up to a reduction of 1024, the eight-wave one).  And where they share it, read from the timeline: up to 240 rows per expert, or while one down matrix has at most 48 MB."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _runner(layers, E, K, h, m, batch, seq, r=0):
    from paper_2604_27085_amd import binding as B, harness as H
    cfg = B.make_cfg(layers, h, 4, 2, 64, m, n_experts=E, top_k=K, lora_rank=r, lora=("q", "o") if r else (), train_base=0)
    s = H.StageRunner(cfg, batch, seq)
    g = torch.Generator(device="cuda:0").manual_seed(h + seq)
    s.slots[0].view(torch.bfloat16).normal_(0.0, 0.05, generator=g)
    x = torch.empty((batch * seq, h), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)
    dy = torch.empty_like(x).normal_(0.0, 1.0, generator=g)
    router = torch.randn((layers, batch * seq, E), generator=g, device="cuda:0")
    torch.cuda.synchronize()
    s.bind()
    return s, x, dy, router


@pytest.mark.parametrize("layers,E,K,h,m,batch,seq", [
    (1, 8, 2, 256, 96, 1, 8),          # experts without rows, a tile column that is not full
    (2, 8, 2, 360, 360, 1, 904),       # experts with one tile and with two; the pair is the last layer's only
    (1, 6, 4, 1032, 520, 3, 232),      # several tile columns, ragged; a reduction beyond 1024 and one within
    (1, 3, 1, 1024, 1032, 1, 40),      # 1024 and 1032
    (1, 24, 2, 1032, 1024, 1, 48),     # the same above 128 MiB of weights: four waves everywhere
])
def test_phases_together_and_apart(layers, E, K, h, m, batch, seq):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B
    s, x, dy, router = _runner(layers, E, K, h, m, batch, seq, r=8)
    outs = []
    for phases in ((B.PHASE_BOTH,), (B.PHASE_RECOMPUTE, B.PHASE_BACKWARD)):
        ws = torch.full((s.wsbytes,), 255, dtype=torch.uint8, device="cuda:0")       # NaN wherever nothing was written
        out, dx, gr, dr = torch.full_like(x, float("nan")), torch.full_like(x, float("nan")), torch.zeros_like(s.grads), torch.full_like(router, float("nan"))
        torch.cuda.synchronize()
        B.rp_trace_start(s.ctx, 512)
        for ph in phases:
            B.rp_stage_backward(s.ctx, 0, ph, x, dy, dx, out if ph & B.PHASE_RECOMPUTE else None, gr, router, dr, batch, seq, ws, s.wsbytes)
        names = [t[0] for t in B.rp_trace_stop(s.ctx, 512)]
        assert names.count("gemm_grouped_pair") == (1 if len(phases) == 1 else 0)
        outs.append((out, dx, gr, dr))
    s.close()
    for a, b in zip(*outs):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)


@pytest.mark.parametrize("m,seq,pair", [(5856, 488, True), (5864, 480, True), (5864, 488, False)])
def test_where_the_pair_is_taken(m, seq, pair):
    """Two experts of 4096 x m: 47.97 and 48.04 MB; 480 rows are 240 per expert."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B
    s, x, dy, router = _runner(1, 2, 1, 4096, m, 1, seq)
    B.rp_trace_start(s.ctx, 512)
    B.rp_stage_backward(s.ctx, 0, B.PHASE_BOTH, x, dy, torch.empty_like(x), None, None, router, None, 1, seq, s.ws, s.wsbytes)
    names = [t[0] for t in B.rp_trace_stop(s.ctx, 512)]
    s.close()
    assert names.count("gemm_grouped_pair") == int(pair)
