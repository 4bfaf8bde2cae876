"""A forward stage in the smallest workspace it accepts: without adapters that holds no scratch for a split of the reduction, so the
products run unsplit.  Against the workspace that rp_query_sizes asks for: fp32 sums in another order, which flips bf16 roundings
(2^-8 each) of a share of the values of every tensor on the way; bound 4e-3."""
import re

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_forward_stage_in_the_smallest_workspace_it_accepts():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h = 264, 1024
    cfg = B.make_cfg(1, h, 8, 2, 128, 3072)
    r = H.StageRunner(cfg, 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    torch.cuda.synchronize()
    r.bind()
    with pytest.raises(B.RpError) as e:
        B.rp_stage_forward(r.ctx, 0, x, torch.empty_like(x), None, None, 1, T, r.ws, 256)
    assert e.value.code == B.RP_ENOMEM
    need = int(re.search(r"< (\d+)", str(e.value)).group(1))
    assert need < r.wsbytes
    outs = []
    for nbytes in (r.wsbytes, r.wsbytes, need):
        ws = torch.full((nbytes + (1 << 20),), 255, dtype=torch.uint8, device="cuda:0")
        out = torch.full_like(x, float("nan"))
        torch.cuda.synchronize()
        B.rp_stage_forward(r.ctx, 0, x, out, None, None, 1, T, ws, nbytes)
        r.sync()
        assert bool((ws[nbytes:] == 255).all())
        outs.append(out)
    r.close()
    assert torch.equal(outs[0], outs[1])
    d = (outs[2].double() - outs[0].double()).norm() / outs[0].double().norm()
    assert 0.0 <= float(d) < 4e-3


@pytest.mark.parametrize("train,rank,experts", [(1, 0, 0), (0, 8, 0), (0, 0, 8)])
def test_every_call_takes_the_least_workspace_and_no_less(train, rank, experts):
    """rp_query_least_workspace names the smallest workspace of each call; against the whole one, bounds as above (2^-8 roundings that
    flip on the way, gradients of a stage through three of them)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, h = 264, 512
    cfg = B.make_cfg(2, h, 8, 2, 128, 512, vocab=0 if experts else 33000, n_experts=experts, top_k=2 if experts else 0, lora_rank=rank,
                     lora=("q", "o") if rank else (), train_base=train)
    r = H.StageRunner(cfg, 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.03)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy = torch.empty_like(x).normal_()
    labels = torch.randint(0, 33000, (T,), dtype=torch.int32, device="cuda:0")
    router = torch.randn((2, T, experts), device="cuda:0") if experts else None
    torch.cuda.synchronize()
    r.bind()
    least = B.rp_query_least_workspace(cfg, 1, T)

    def forward(ws, n):
        out = torch.full_like(x, float("nan"))
        torch.cuda.synchronize()
        B.rp_stage_forward(r.ctx, 0, x, out, None, router, 1, T, ws, n)
        return [out]

    def backward(ws, n):
        dx, gr = torch.full_like(x, float("nan")), torch.zeros_like(r.grads)
        torch.cuda.synchronize()
        B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, gr if r.gbytes else None, router, None, 1, T, ws, n)
        return [dx, gr] if r.gbytes else [dx]

    def head(ws, n):
        dx, loss, gr = torch.full_like(x, float("nan")), torch.zeros(1, device="cuda:0"), torch.zeros_like(r.grads)
        torch.cuda.synchronize()
        B.rp_lmhead_ce_fwd_bwd(r.ctx, 0, x, labels, loss, dx, gr if train else None, 1.0, 1, T, ws, n)
        return [dx, loss, gr] if train else [dx, loss]

    for call, need in zip((forward, backward, head), least):
        if need == 0:
            continue
        outs = []
        for nbytes in (r.wsbytes, need):
            ws = torch.full((nbytes + (1 << 20),), 255, dtype=torch.uint8, device="cuda:0")
            outs.append(call(ws, nbytes))
            r.sync()
            assert bool((ws[nbytes:] == 255).all())
        with pytest.raises(B.RpError) as e:
            call(r.ws, need - 1)
        assert e.value.code == B.RP_ENOMEM
        for a, b in zip(*outs):
            assert float((a.double() - b.double()).norm() / a.double().norm()) < 8e-3
    r.close()
