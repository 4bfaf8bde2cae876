"""The SwiGLU arithmetic at every finite bf16 gate value, against 64 bits.  The kernels take exp(-g) with the hardware exponential
(relative error |g| 2^-24 from rounding its argument, 6e-6 at the end of the range, plus an ulp), divide, and round to bf16
(2^-8).  exp(-g) overflows below g = -88.72: the results are zeros there."""
import numpy as np
import pytest

from test_gpu_kernels import dev, stream

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_swiglu_at_every_gate_value():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    T, m = 16, 4096
    g = (np.arange(65536, dtype=np.uint32) << 16).view(np.float32).reshape(T, m)
    g = np.where(np.isfinite(g), g, np.float32(0))
    gu = dev(H, np.concatenate([g, np.ones_like(g)], axis=1))
    act = torch.empty((T, m), dtype=torch.bfloat16, device="cuda:0")
    dgu = torch.empty((T, 2 * m), dtype=torch.bfloat16, device="cuda:0")
    B.rp_op_swiglu_fwd(stream(), gu, act, T, m)
    B.rp_op_swiglu_bwd(stream(), torch.ones_like(act), gu, dgu, T, m)
    torch.cuda.synchronize()
    a, dg, du = (H.to_f32(t).astype(np.float64) for t in (act, dgu[:, :m], dgu[:, m:]))
    x = g.astype(np.float64)
    with np.errstate(over="ignore"):
        s = 1.0 / (1.0 + np.exp(-x))
    rest = -np.expm1(-np.logaddexp(0.0, -x))          # 1 - s without cancellation
    over = x < -88.72
    assert not (a[over].any() or dg[over].any() or du[over].any())
    tiny = 2.0 ** -133                                # spacing of the subnormal bf16 numbers
    rel = 2.0 ** -8 + 1e-5
    for name, got in (("act", a), ("d up", du)):
        bad = ~over & (np.abs(got - x * s) > rel * np.abs(x * s) + tiny)
        assert not bad.any(), (name, g[bad][:8])
    # d gate = s (1 + g (1 - s)): the error of s moves both factors, 1 - s loses up to 2^-25 against g <= 17
    ref = s * (1.0 + x * rest)
    bad = ~over & (np.abs(dg - ref) > rel * np.abs(ref) + 2e-5 * s * rest * (1.0 + np.abs(x)) + 2e-6 * s + tiny)
    assert not bad.any(), ("d gate", g[bad][:8])
