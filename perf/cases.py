"""What the speed of the worker hot path is measured on.

A case is one call sequence that a worker process makes, on inputs that are already on the GPU:

  fwd    rp_stage_forward     a forward stage (its output and, with a router in the layer, the router logits)
  bwd    rp_stage_backward    a backward stage with recomputation: stage output, input gradient, weight gradients
  fused  the fused last stage (recompute -> LM head + loss -> backward), as harness.StageRunner.fused_last_stage runs it
  head   rp_lmhead_ce_fwd_bwd on a stage that is the LM head alone: loss, input gradient, weight gradients
  attn   rp_op_attn_fwd followed by rp_op_attn_bwd: output, log-sum-exp, dq, dk, dv

Weight gradients accumulate in place, so a pass of a kind that has them starts by clearing the gradient blob, as the first
micro-batch of a training step does.  The layer shapes are those of synth.CONFIGS.  Weights are drawn straight into the device
slot and bound with rp_stage_bind_weights: the upload is a host-link copy that overlaps the stage and has no case here.
"""
import math

import torch

import synth
from paper_2604_27085_amd import binding as B
from paper_2604_27085_amd import harness as H

DEV = "cuda:0"
F64 = torch.float64
BF16 = torch.bfloat16
LORA = {"q": "q", "k": "k", "v": "v", "o": "o", "g": "gate", "u": "up", "d": "down"}     # letters of a case's "lora"


def _shape(name, **over):
    """The plain values of one synth configuration; `over` replaces some of them."""
    c = synth.CONFIGS[name]
    letters = {v: k for k, v in LORA.items()}
    out = dict(layers=1, h=c["hidden"], a=c["n_q_heads"], kh=c["n_kv_heads"], d=c["head_dim"], m=c["ffn"], V=0, E=c["n_experts"],
               topk=c["top_k"], r=c["lora_rank"], lora="".join(letters[n] for n in c["lora"]), train=c["train_base"],
               router=c.get("moe_router", 0), batch=1, seq=c["seq"])
    out.update(over)
    return out


def listed():
    return [
        # the smallest training step anybody runs: a toy model in a test or a smoke run; launches and latency
        dict(name="fused_toy_128", kind="fused", **_shape("C1", layers=2, V=4096, seq=128)),
        # a forward stage on a short prompt of a length that fills no tile
        dict(name="fwd_short_1000", kind="fwd", **_shape("C2", seq=1000)),
        # LoRA fine-tuning on short instruction data: two sequences of 508 tokens, adapters on all projections
        dict(name="bwd_lora_2x508", kind="bwd", **_shape("C3", batch=2, seq=508)),
        # mid-sized forward stage: a batch of four ordinary sequences through two layers
        dict(name="fwd_4x1024", kind="fwd", **_shape("C3", layers=2, r=0, lora="", batch=4, seq=1024)),
        # full fine-tuning of a small model at the sequence length it is usually trained with
        dict(name="bwd_full_4096", kind="bwd", **_shape("C2")),
        # LoRA fine-tuning of a mid-sized and of a large model on long sequences; the second is the largest case
        dict(name="bwd_lora_8192", kind="bwd", **_shape("C3")),
        dict(name="bwd_lora_16384", kind="bwd", **_shape("C4")),
        # mixture of experts: forward with the router in the layer; backward with few tokens per expert
        dict(name="fwd_moe_8192", kind="fwd", **_shape("C6")),
        dict(name="bwd_moe_2048", kind="bwd", **_shape("C5", seq=2048)),
        # the oversized last stage: trainable head of the small model, frozen head of the large one on a short ragged batch
        dict(name="head_train_4096", kind="head", **_shape("C2", layers=0, V=151936)),
        dict(name="head_frozen_2040", kind="head", **_shape("C4", layers=0, V=151936, r=0, lora="", seq=2040)),
        # the attention kernels alone, forward and backward, at head dimension 64 and a length that fills no tile
        dict(name="attn_d64_3x1500", kind="attn", **_shape("C6", batch=3, seq=1500)),
    ]


# (kind, configuration, overrides, shortest, longest): tokens of a drawn case
_DRAWS = [
    ("fused", "C1", dict(layers=2, V=4096), 64, 2048),
    ("fwd", "C1", {}, 64, 4096),
    ("fwd", "C2", {}, 64, 8192),
    ("bwd", "C2", {}, 64, 8192),
    ("fwd", "C3", {}, 64, 8192),
    ("bwd", "C3", {}, 64, 8192),
    ("fwd", "C4", {}, 128, 8192),
    ("bwd", "C4", {}, 128, 8192),
    ("bwd", "C3", dict(r=0, lora="", train=1), 64, 4096),
    ("fwd", "C6", {}, 128, 8192),
    ("bwd", "C6", {}, 128, 8192),
    ("bwd", "C5", {}, 128, 8192),
    ("head", "C2", dict(layers=0, V=151936), 64, 4096),
    ("head", "C4", dict(layers=0, V=151936, r=0, lora=""), 64, 4096),
    ("attn", "C2", {}, 128, 8192),
    ("attn", "C3", {}, 128, 8192),
    ("attn", "C6", {}, 128, 8192),
]


def draw(rng):
    kind, name, over, lo, hi = rng.choice(_DRAWS)
    batch = rng.choice((1, 1, 1, 2, 3, 4))
    tokens = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    step = 8 // math.gcd(batch, 8)                      # batch * seq is a multiple of 8
    seq = max(1, round(tokens / batch / step)) * step
    return dict(kind=kind, **_shape(name, batch=batch, seq=seq, **over))


# ---------------------------------------------------------------------------------------------------- inputs
def _lora_names(case):
    return [LORA[x] for x in case["lora"]] if case["r"] else []


def _dims(case):
    return case["a"] * case["d"], case["kh"] * case["d"]


def _tensor_shapes(case):
    """(blob name, shape, standard deviation, mean) of every tensor of a layer, in the blob's order; then the head's."""
    h, d, m, E, r = case["h"], case["d"], case["m"], case["E"], case["r"]
    qd, kd = _dims(case)
    lay = [("G1", (h,), 0.1, 1.0), ("WQKV", (qd + 2 * kd, h), 0.02, 0.0), ("GQ", (d,), 0.1, 1.0), ("GK", (d,), 0.1, 1.0),
           ("WO", (h, qd), 0.02, 0.0), ("G2", (h,), 0.1, 1.0),
           ("WGU", (E, 2 * m, h) if E else (2 * m, h), 0.02, 0.0), ("WD", (E, h, m) if E else (h, m), 0.02, 0.0)]
    if case["router"]:
        lay.append(("WR", (E, h), 0.002, 0.0))
    ins = {"q": (qd, h), "k": (kd, h), "v": (kd, h), "o": (h, qd), "gate": (m, h), "up": (m, h), "down": (h, m)}
    for n in _lora_names(case):
        lay.append(("LA_" + n.upper(), (r, ins[n][1]), 0.02, 0.0))
        lay.append(("LB_" + n.upper(), (ins[n][0], r), 0.01, 0.0))
    head = [("GF", (h,), 0.1, 1.0), ("WV", (case["V"], h), 0.02, 0.0)] if case["V"] else []
    return lay, head


def _draw_tensors(case, seed):
    """Yields (layer, blob name, bf16 tensor) for all weights, then the activations, always in the same order from one
    generator, so that prepare() and exact() see the same numbers."""
    g = torch.Generator(device=DEV).manual_seed(seed)

    def normal(shape, std, mean=0.0):
        t = torch.empty(shape, dtype=BF16, device=DEV)
        t.normal_(mean, std, generator=g)
        return t

    T, h, E = case["batch"] * case["seq"], case["h"], case["E"]
    lay, head = _tensor_shapes(case)
    x = normal((T, h), 1.0)
    if case["router"]:
        # a trained router is decisive: every token has top-k planted coordinates, which its experts' rows pick up
        x[:, :E] *= 0.5
        pick = torch.rand(T, E, generator=g, device=DEV).argsort(1)[:, :case["topk"]]
        x.scatter_(1, pick, (8.0 + 2.0 * torch.arange(case["topk"], device=DEV)).to(BF16).expand(T, -1).contiguous())
    yield None, "x", x
    yield None, "dy", normal((T, h), 1.0)
    if E and not case["router"]:
        yield None, "logits", torch.randn((max(case["layers"], 1), T, E), generator=g, device=DEV)
    if case["V"]:
        lab = torch.randint(0, case["V"], (case["batch"], case["seq"]), generator=g, device=DEV, dtype=torch.int32)
        lab[:, -1] = B.IGNORE_INDEX                      # the last token of a sequence has no successor
        yield None, "labels", lab.reshape(-1)
    for layer, tensors in [(i, lay) for i in range(case["layers"])] + [(case["layers"], head)]:
        for name, shape, std, mean in tensors:
            t = normal(shape, std, mean)
            if name == "WR":
                t[torch.arange(E, device=DEV), torch.randperm(E, generator=g, device=DEV)] = 0.25
            yield layer, name, t


class _Stage:
    """A worker's context, bound weights and buffers for one stage shape."""

    def __init__(self, case, seed):
        T, h = case["batch"] * case["seq"], case["h"]
        cfg = B.make_cfg(case["layers"], h, case["a"], case["kh"], case["d"], case["m"], vocab=case["V"], n_experts=case["E"],
                         top_k=case["topk"], lora_rank=case["r"], lora=_lora_names(case), train_base=case["train"],
                         moe_router=case["router"])
        self.case, self.r = case, H.StageRunner(cfg, case["batch"], case["seq"], device=DEV)
        self.inp, slot = {}, self.r.slots[0].view(BF16)
        for layer, name, t in _draw_tensors(case, seed):
            if layer is None:
                self.inp[name] = t
                continue
            off, n = B.rp_weight_layout(cfg, layer, B.T[name])
            assert n == t.numel(), (name, n, tuple(t.shape))
            slot[off // 2:off // 2 + n] = t.reshape(-1)
        torch.cuda.synchronize()
        self.r.bind()
        bf = lambda: torch.empty((T, h), dtype=BF16, device=DEV)  # noqa: E731
        self.out, self.dx, self.dy_head = bf(), bf(), bf()
        self.loss = torch.empty(1, dtype=torch.float32, device=DEV)
        self.router = self.inp.get("logits")
        if case["router"]:
            self.router = torch.empty((case["layers"], T, case["E"]), dtype=torch.float32, device=DEV)
        self.d_router = torch.empty_like(self.router) if self.router is not None else None
        self.grads = {}
        lay, head = _tensor_shapes(case)
        for layer, tensors in [(i, lay) for i in range(case["layers"])] + [(case["layers"], head)]:
            for name, shape, _, _ in tensors:
                off, n = B.rp_grad_layout(cfg, layer, B.T[name])
                if n:
                    self.grads["%d.%s" % (layer, name)] = self.r.grads[off // 4:off // 4 + n].view(shape)
        torch.cuda.synchronize()

    def __del__(self):
        if getattr(self, "r", None) is not None:
            self.r.close()

    def clear_grads(self):
        if self.r.gbytes:
            with torch.cuda.stream(self.r.compute):
                self.r.grads.zero_()


class _Attention:
    """q, k, v and the output gradient of one attention layer, with the outputs and scratch the kernels take."""

    def __init__(self, case, seed):
        g = torch.Generator(device=DEV).manual_seed(seed)
        T, a, kh, d = case["batch"] * case["seq"], case["a"], case["kh"], case["d"]
        mk = lambda n: torch.empty((T, n, d), dtype=BF16, device=DEV)  # noqa: E731
        self.case = case
        self.q, self.k, self.v, self.do = [t.normal_(0.0, 1.0, generator=g) for t in (mk(a), mk(kh), mk(kh), mk(a))]
        self.o, self.dq, self.dk, self.dv = mk(a), mk(a), mk(kh), mk(kh)
        self.lse = torch.empty((case["batch"], a, case["seq"]), dtype=torch.float32, device=DEV)
        self.delta = torch.empty_like(self.lse)
        self.scratch = torch.empty((2, T, a, d), dtype=torch.float32, device=DEV)


def prepare(case, seed):
    return _Attention(case, seed) if case["kind"] == "attn" else _Stage(case, seed)


# ---------------------------------------------------------------------------------------------------- one pass
def _run_attention(s):
    c = s.case
    st = torch.cuda.current_stream().cuda_stream
    b, n, a, kh, d = c["batch"], c["seq"], c["a"], c["kh"], c["d"]
    qd, kd = _dims(c)
    B.rp_op_attn_fwd(st, s.q, s.k, s.v, s.o, s.lse, qd, kd, kd, qd, b, n, a, kh, d)
    B.rp_op_attn_bwd(st, s.q, s.k, s.v, s.o, s.do, s.lse, s.delta, s.dq, s.dk, s.dv, s.scratch, qd, kd, kd, qd, qd, qd, kd, kd,
                     b, n, a, kh, d)
    return {"o": s.o, "lse": s.lse, "dq": s.dq, "dk": s.dk, "dv": s.dv}


def run(state):
    s, c = state, state.case
    if c["kind"] == "attn":
        return _run_attention(s)
    r, x = s.r, s.inp["x"]
    if c["kind"] == "fwd":
        B.rp_stage_forward(r.ctx, 0, x, s.out, None, s.router, r.batch, r.seq, r.ws, r.wsbytes)
        return {"out": s.out, "router": s.router if c["router"] else None}
    s.clear_grads()
    if c["kind"] == "bwd":
        B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, s.inp["dy"], s.dx, s.out, r.grads if r.gbytes else None, s.router, s.d_router,
                            r.batch, r.seq, r.ws, r.wsbytes)
        return {"out": s.out, "dx": s.dx, "grads": s.grads, "router": s.router if c["router"] else None, "d_router": s.d_router}
    if c["kind"] == "head":
        r.head(x, s.inp["labels"], train=bool(c["train"]), loss=s.loss, dx=s.dx)
        return {"loss": s.loss, "dx": s.dx, "grads": s.grads}
    r.fused_last_stage(x, s.inp["labels"], s.out, s.dy_head, s.dx, s.loss)
    return {"out": s.out, "loss": s.loss, "dx": s.dx, "grads": s.grads}


# ---------------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    """Projections 2*T*N*K each: once forward, once more for the input gradient, once more for a weight gradient; causal
    attention 2*s^2*a*d per sequence forward and 2.5 times that backward; the LM head 2*T*h*V per product, three when it
    trains, two when it is frozen.  Bytes: weights, inputs and outputs once each (fp32 gradients written once)."""
    c, kind = case, case["kind"]
    T, h, m, E, r = c["batch"] * c["seq"], c["h"], c["m"], c["E"], c["r"]
    qd, kd = _dims(c)
    s2 = 2.0 * c["batch"] * c["seq"] * c["seq"] * qd
    if kind == "attn":
        return {"flops": 3.5 * s2, "bytes": 2.0 * T * (4 * qd + 4 * kd) + 4.0 * T * c["a"]}
    lay, head = _tensor_shapes(c)
    count = lambda ts: sum(math.prod(shape) for _, shape, _, _ in ts)  # noqa: E731
    lora = count([t for t in lay if t[0][:3] in ("LA_", "LB_")])
    backward = kind in ("bwd", "fused")
    proj = 2.0 * T * (h * (qd + 2 * kd) + qd * h + (E * h if c["router"] else 0)) + 2.0 * T * (c["topk"] if E else 1) * 3 * h * m
    products = (2.0 + c["train"]) if backward else 1.0
    flops = c["layers"] * (proj * products + 2.0 * T * lora * (3.0 if backward else 1.0) + s2 * (3.5 if backward else 1.0))
    # the experts that some token chose have to be read: all of them, unless there are fewer choices than experts
    used = min(1.0, T * c["topk"] / E) if E else 1.0
    experts = count([t for t in lay if t[0] in ("WGU", "WD")]) if E else 0
    nbytes = c["layers"] * 2.0 * (count(lay) - (1.0 - used) * experts) + 2.0 * T * h * 2
    nbytes += 4.0 * c["layers"] * T * E
    if backward:
        nbytes += 2.0 * T * h * 2 + c["layers"] * 4.0 * (count(lay) if c["train"] else lora) + 4.0 * c["layers"] * T * E
    if c["V"]:
        flops += (4.0 + 2.0 * c["train"]) * T * h * c["V"]
        nbytes += 2.0 * count(head) + 4.0 * T + (4.0 * count(head) if c["train"] else 0.0)
    return {"flops": flops, "bytes": nbytes}


def tolerance(case):
    """bf16 storage of every intermediate: two correct implementations round the same tensors differently.  Measured distance
    to 64-bit results: attention 2.5e-3, forward stages and heads 2e-3 to 7e-3, backward stages up to 8.5e-3 (the gradients of
    the q/k path, where four rounded factors meet)."""
    return {"rel": 2e-2 if case["kind"] in ("bwd", "fused") else 1e-2}


# ---------------------------------------------------------------------------------------------------- 64-bit definition
def _rms(x, g, eps=1.0e-6):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g


class _CausalAttention(torch.autograd.Function):
    """Causal attention of [batch, seq, heads, d] tensors with grouped queries, one head at a time."""

    @staticmethod
    def _probs(q, k):
        s = (q @ k.t()) / math.sqrt(q.shape[1])
        s.masked_fill_(torch.ones(s.shape, dtype=torch.bool, device=s.device).triu_(1), -math.inf)
        lse = torch.logsumexp(s, 1)
        return s.sub_(lse[:, None]).exp_(), lse

    @staticmethod
    def forward(ctx, q, k, v):
        o = torch.empty_like(q)
        lse = torch.empty((q.shape[0], q.shape[2], q.shape[1]), dtype=q.dtype, device=q.device)
        grp = q.shape[2] // k.shape[2]
        for b in range(q.shape[0]):
            for i in range(q.shape[2]):
                p, lse[b, i] = _CausalAttention._probs(q[b, :, i].contiguous(), k[b, :, i // grp].contiguous())
                o[b, :, i] = p @ v[b, :, i // grp].contiguous()
        ctx.save_for_backward(q, k, v, o)
        ctx.mark_non_differentiable(lse)
        return o, lse

    @staticmethod
    def backward(ctx, do, _):
        q, k, v, o = ctx.saved_tensors
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        grp = q.shape[2] // k.shape[2]
        for b in range(q.shape[0]):
            for i in range(q.shape[2]):
                qi, ki, vi = q[b, :, i].contiguous(), k[b, :, i // grp].contiguous(), v[b, :, i // grp].contiguous()
                di = do[b, :, i].contiguous()
                p, _ = _CausalAttention._probs(qi, ki)
                dv[b, :, i // grp] += p.t() @ di
                ds = (di @ vi.t()).sub_((di * o[b, :, i]).sum(1, keepdim=True)).mul_(p).div_(math.sqrt(q.shape[3]))
                dq[b, :, i] = ds @ ki
                dk[b, :, i // grp] += ds.t() @ qi
        return dq, dk, dv


def _rope(x):
    """x [batch, seq, heads, d]: pairs (i, i + d/2) turned by pos * 1e6^(-2i/d)."""
    n, d = x.shape[1], x.shape[3]
    ang = torch.arange(n, dtype=F64, device=DEV)[:, None] * 1.0e6 ** (-torch.arange(0, d, 2, dtype=F64, device=DEV) / d)
    co, si = ang.cos()[:, None], ang.sin()[:, None]
    x1, x2 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat((x1 * co - x2 * si, x2 * co + x1 * si), -1)


def _layer(case, w, x, logits):
    b, n, h, d, m = case["batch"], case["seq"], case["h"], case["d"], case["m"]
    qd, kd = _dims(case)

    def adapter(name, t):
        return (t @ w["LA_" + name].t()) @ w["LB_" + name].t() if "LA_" + name in w else 0.0

    n1 = _rms(x, w["G1"])
    q, k, v = (n1 @ w["WQKV"].t()).split((qd, kd, kd), 1)
    q, k, v = q + adapter("Q", n1), k + adapter("K", n1), v + adapter("V", n1)
    q = _rope(_rms(q.reshape(b, n, case["a"], d), w["GQ"]))
    k = _rope(_rms(k.reshape(b, n, case["kh"], d), w["GK"]))
    o = _CausalAttention.apply(q, k, v.reshape(b, n, case["kh"], d))[0].reshape(b * n, qd)
    y = x + o @ w["WO"].t() + adapter("O", o)
    n2 = _rms(y, w["G2"])
    if not case["E"]:
        g, u = (n2 @ w["WGU"].t()).split(m, 1)
        act = torch.nn.functional.silu(g + adapter("GATE", n2)) * (u + adapter("UP", n2))
        return y + act @ w["WD"].t() + adapter("DOWN", act), None
    if case["router"]:
        logits = n2 @ w["WR"].t()
    top = logits.topk(case["topk"], 1)
    p = top.values.softmax(1)
    z = y
    for e in range(case["E"]):
        t, j = (top.indices == e).nonzero(as_tuple=True)
        if t.numel() == 0:
            continue
        gu = n2[t] @ w["WGU"][e].double().t()
        act = torch.nn.functional.silu(gu[:, :m]) * gu[:, m:]
        z = z.index_add(0, t, (act @ w["WD"][e].double().t()) * p[t, j, None])
    return z, logits


def exact(case, seed):
    if case["kind"] == "attn":
        s = _Attention(case, seed)
        sh = lambda t: t.double().reshape(case["batch"], case["seq"], t.shape[1], case["d"])  # noqa: E731
        q, k, v = [sh(t).requires_grad_() for t in (s.q, s.k, s.v)]
        o, lse = _CausalAttention.apply(q, k, v)
        g = torch.autograd.grad(o, (q, k, v), sh(s.do))
        flat = lambda t: t.detach().reshape(-1, t.shape[2], case["d"])  # noqa: E731
        return {"o": flat(o), "lse": lse, "dq": flat(g[0]), "dk": flat(g[1]), "dv": flat(g[2])}
    inp, w = {}, {}
    for layer, name, t in _draw_tensors(case, seed):
        if layer is None:
            inp[name] = t
        else:      # the experts' weights are widened one expert at a time
            w.setdefault(layer, {})[name] = t if t.dim() == 3 else t.double()
    want = {}
    for layer, ts in w.items():
        for name, t in ts.items():
            if name[:3] in ("LA_", "LB_") or case["train"]:
                want["%d.%s" % (layer, name)] = t.requires_grad_()
    x = inp["x"].double().requires_grad_()
    given = inp["logits"].double().requires_grad_() if "logits" in inp else None
    z, logits = x, []
    with torch.set_grad_enabled(case["kind"] != "fwd"):
        for i in range(case["layers"]):
            z, lg = _layer(case, w[i], z, given[i] if given is not None else None)
            logits.append(lg)
        out, loss = z, None
        if case["V"]:
            hw = w[case["layers"]]
            zl = _rms(z, hw["GF"]) @ hw["WV"].t()
            lab = inp["labels"].long()
            loss = torch.nn.functional.cross_entropy(zl, lab, ignore_index=B.IGNORE_INDEX).reshape(1)
    router = torch.stack([t.detach() for t in logits]) if case["router"] else None
    if case["kind"] == "fwd":
        return {"out": out.detach(), "router": router}
    wrt = [x] + list(want.values())
    if case["E"]:
        wrt += [given] if given is not None else logits
    g = torch.autograd.grad(loss if case["V"] else out, wrt, None if case["V"] else inp["dy"].double())
    grads = dict(zip(want, g[1:1 + len(want)]))
    if case["kind"] == "head":
        return {"loss": loss.detach(), "dx": g[0], "grads": grads}
    if case["kind"] == "fused":
        return {"out": out.detach(), "loss": loss.detach(), "dx": g[0], "grads": grads}
    d_router = None
    if case["E"]:
        rest = g[1 + len(want):]
        d_router = rest[0] if given is not None else torch.stack(rest)
    return {"out": out.detach(), "dx": g[0], "grads": grads, "router": router, "d_router": d_router}
