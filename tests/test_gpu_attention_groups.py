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
    (1, 128, 4, 2, 64),       # both of two: one key tile
    (4, 256, 16, 8, 128),     # both of two: two key tiles and 64 heads in all
    (3, 256, 20, 10, 64),     # one of two: 60
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


@pytest.mark.parametrize("d", [64, 128])
def test_backward_in_place(d):
    """dq in the place of q or of the output's gradient: delta comes from a kernel of its own and dQ last, with the same result but
    for the rounding of delta's sum (2^-24 of each term, far below the bf16 step of dS)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B
    b, n, a, kh = 2, 200, 4, 2
    g = torch.Generator(device="cuda:0").manual_seed(5)
    mk = lambda k: torch.empty((b * n, k, d), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)  # noqa: E731
    q, k, v, do = mk(a), mk(kh), mk(kh), mk(a)
    o, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    lse = torch.empty((b, a, n), dtype=torch.float32, device="cuda:0")
    scratch = torch.empty((2, b * n, a, d), dtype=torch.float32, device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    B.rp_op_attn_fwd(st, q, k, v, o, lse, a * d, kh * d, kh * d, a * d, b, n, a, kh, d)
    want = None
    for place in ("own", "q", "do"):
        q1, do1, delta = q.clone(), do.clone(), torch.full_like(lse, float("nan"))
        dq = dict(own=torch.empty_like(q), q=q1, do=do1)[place]
        B.rp_op_attn_bwd(st, q1, k, v, o, do1, lse, delta, dq, dk, dv, scratch, a * d, kh * d, kh * d, a * d, a * d, a * d, kh * d, kh * d,
                         b, n, a, kh, d)
        torch.cuda.synchronize()
        got = [t.double().clone() for t in (dq, dk, dv, delta)]
        ref = (do.double() * o.double()).sum(-1).view(b, n, a).transpose(1, 2)
        assert float((got[3] - ref).norm() / ref.norm()) < 1e-6
        want = want or got
        for x, y in zip(got[:3], want):
            assert float((x - y).norm() / y.norm()) < 1e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("place", ["o, from row 9 on", "scratch", "end of scratch", "beside q"])
def test_backward_with_dq_in_memory_that_is_free_by_then(d, place):
    """dq inside o at another offset, inside scratch (both free when delta and the partials have been used), and in columns beside q of
    one array: the same results as in memory of its own but for delta's rounding, as above."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B
    b, n, a, kh = 2, 264, 4, 2
    T, w = b * n, a * d
    g = torch.Generator(device="cuda:0").manual_seed(6)
    mk = lambda k: torch.empty((T, k * d), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 1.0, generator=g)  # noqa: E731
    q, k, v, do = mk(a), mk(kh), mk(kh), mk(a)
    lse = torch.empty((b, a, n), dtype=torch.float32, device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    got = []
    for where in ("own", place):
        scratch = torch.full((2 * T * w,), float("nan"), dtype=torch.float32, device="cuda:0")
        room = torch.zeros((T + 9, w), dtype=torch.bfloat16, device="cuda:0")
        both = torch.cat((q, torch.zeros_like(q)), 1)
        o, dk, dv, delta = room[:T], torch.empty_like(k), torch.empty_like(v), torch.empty_like(lse)
        half = scratch.view(torch.bfloat16).view(-1, w)
        q1, ldq = (both, 2 * w) if where == "beside q" else (q, w)
        dq, lddq = {"own": (torch.empty_like(q), w), "scratch": (half[:T], w), "end of scratch": (half[-T:], w),
                    "o, from row 9 on": (room[9:], w), "beside q": (both[:, w:], 2 * w)}[where]
        B.rp_op_attn_fwd(st, q1, k, v, o, lse, ldq, kh * d, kh * d, w, b, n, a, kh, d)
        B.rp_op_attn_bwd(st, q1, k, v, o, do, lse, delta, dq, dk, dv, scratch, ldq, kh * d, kh * d, w, w, lddq, kh * d, kh * d, b, n, a, kh, d)
        torch.cuda.synchronize()
        got.append([t.double().clone() for t in (dq, dk, dv)])
    for x, y in zip(got[1], got[0]):
        assert float((x - y).norm() / y.norm()) < 1e-3
