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
