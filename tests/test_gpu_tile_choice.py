"""The tile that a stage's products take, from the timeline: 256x256 only where more than half of the CUs get one, since a worker's calls run one
after the other on one stream and nothing else fills the rest (whatever the reduction, and whichever of its kernels would run)."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (tokens, hidden, query heads of 64, ffn): outputs of tokens x hidden in 128, 128 (ragged) and 144 tiles of 256x256
@pytest.mark.parametrize("T,h,a,m,big", [
    (2048, 4096, 40, 4096, False),      # reductions of 2560, 4096, 8192, 7680
    (4088, 2040, 16, 6144, False),      # of 1024, 6144, 12288, 3072
    (2304, 4096, 40, 4096, True),
])
def test_256x256_tiles_where_they_fill_more_than_half_of_the_chip(T, h, a, m, big):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_27085_amd import binding as B, harness as H
    r = H.StageRunner(B.make_cfg(1, h, a, a, 64, m, lora_rank=0, lora=(), train_base=0), 1, T)
    r.slots[0].view(torch.bfloat16).normal_(0.0, 0.02)
    x = torch.empty((T, h), dtype=torch.bfloat16, device="cuda:0").normal_()
    dy, dx = torch.empty_like(x).normal_(), torch.empty_like(x)
    torch.cuda.synchronize()
    r.bind()
    B.rp_trace_start(r.ctx, 256)
    B.rp_stage_backward(r.ctx, 0, B.PHASE_BOTH, x, dy, dx, None, None, None, None, 1, T, r.ws, r.wsbytes)
    rec = B.rp_trace_stop(r.ctx, 256)
    r.close()
    # o and down; the gradients of the inputs of gate | up and of q | k | v
    for layout, K in (("NT", a * 64), ("NT", m), ("NN", 2 * m), ("NN", 3 * a * 64)):
        names = [t[0] for t in rec if t[0].startswith("gemm_") and t[0].endswith(layout) and t[1] == 2.0 * T * h * K]
        assert len(names) == 1 and names[0].startswith("gemm_256x256_") == big, (layout, K, names)
