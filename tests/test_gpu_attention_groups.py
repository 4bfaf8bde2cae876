"""dK/dV workgroups that take several query heads of a group: one, two and four heads, a whole group (no partials), lengths that end
inside a key tile and a query tile.  Against plain attention in fp32; bound: bf16 rounding of the result and of the two operands P and
dS of the products, three independent relative errors of 2^-9 = 2e-3 -> 3.4e-3, bound 5e-3."""
import math

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("batch,seq,a,kh,d", [
    (24, 300, 64, 8, 64),     # four heads of eight per workgroup
    (16, 300, 64, 8, 64),     # two of eight
    (16, 70, 16, 8, 64),      # one of two
    (16, 300, 32, 4, 128),    # four of eight
    (8, 300, 32, 4, 128),     # two of eight
    (32, 300, 16, 4, 128),    # the whole group of four
    (16, 330, 32, 16, 128),   # the whole group of two
    (2, 129, 8, 8, 128),      # no groups
])
def test_heads_per_workgroup(batch, seq, a, kh, d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B
    g = torch.Generator(device="cuda:0").manual_seed(batch * 1000 + seq)
    mk = lambda n: torch.empty((batch * seq, n, d), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)  # noqa: E731
    q, k, v, do = mk(a), mk(kh), mk(kh), mk(a)
    out = [torch.full_like(t, float("nan")) for t in (q, q, k, v)]
    o, dq, dk, dv = out
    lse = torch.empty((batch, a, seq), dtype=torch.float32, device="cuda:0")
    delta = torch.empty_like(lse)
    scratch = torch.full((2, batch * seq, a, d), float("nan"), dtype=torch.float32, device="cuda:0") if a != kh else None
    st = torch.cuda.current_stream().cuda_stream
    runs = []
    for _ in range(2):
        B.rp_op_attn_fwd(st, q, k, v, o, lse, a * d, kh * d, kh * d, a * d, batch, seq, a, kh, d)
        B.rp_op_attn_bwd(st, q, k, v, o, do, lse, delta, dq, dk, dv, scratch, a * d, kh * d, kh * d, a * d, a * d, a * d, kh * d, kh * d,
                         batch, seq, a, kh, d)
        torch.cuda.synchronize()
        runs.append([t.clone() for t in out])
    assert all(torch.equal(x, y) for x, y in zip(*runs))        # sums in a fixed order
    mask = torch.ones((seq, seq), dtype=torch.bool, device="cuda:0").triu(1)
    err = [0.0] * 4
    nrm = [0.0] * 4
    for b in range(batch):
        rows = slice(b * seq, (b + 1) * seq)
        for j in range(kh):
            kj, vj = k[rows, j].float().contiguous(), v[rows, j].float().contiguous()
            dkj, dvj = torch.zeros_like(kj), torch.zeros_like(vj)
            for i in range(j * (a // kh), (j + 1) * (a // kh)):
                qi, di = q[rows, i].float().contiguous(), do[rows, i].float().contiguous()
                p = torch.softmax((qi @ kj.t() / math.sqrt(d)).masked_fill(mask, -math.inf), 1)
                oi = p @ vj
                ds = p * (di @ vj.t() - (di * oi).sum(1, keepdim=True)) / math.sqrt(d)
                dkj += ds.t() @ qi
                dvj += p.t() @ di
                for n, (x, y) in enumerate(((o[rows, i], oi), (dq[rows, i], ds @ kj))):
                    err[n] += float((x.float() - y).square().sum())
                    nrm[n] += float(y.square().sum())
            for n, (x, y) in ((2, (dk[rows, j], dkj)), (3, (dv[rows, j], dvj))):
                err[n] += float((x.float() - y).square().sum())
                nrm[n] += float(y.square().sum())
    for n, name in enumerate(("o", "dq", "dk", "dv")):
        assert math.sqrt(err[n] / nrm[n]) < 5e-3, name
