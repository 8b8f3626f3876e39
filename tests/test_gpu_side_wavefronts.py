"""Recurrences whose workgroups have wavefronts of their own for what is not the exchange, four frames ahead: few frames, widths and
batches at the edges of slices, tiles and built widths, z written by the recurrence, exchange copies marked by it."""
import pytest

from test_gpu_parity import check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,H", [
    (1, 1, 8), (2, 16, 8), (3, 17, 24), (5, 50, 320),       # H below a slice, one frame, every remainder of four frames
    (4, 64, 512), (6, 49, 392), (7, 128, 256), (5, 200, 128),   # eight groups and more, through the L2
    (3, 33, 512), (2, 8, 768), (5, 15, 776), (4, 30, 1024), (9, 20, 640),   # one look, two halves of the operand
])
def test_few_sequences_bf16(T, B, H):
    check_step(dict(T=T, B=B, D=8, H=H, L=2, P=0, V=20), 1, seed=95, theta_scale=1.0 if H > 500 else 2.0)


@pytest.mark.parametrize("T,B,H", [
    (2, 1, 1), (3, 17, 30), (4, 33, 33), (5, 16, 16), (9, 8, 32),
    (2, 64, 512), (3, 20, 513), (4, 33, 384), (5, 40, 130),     # backward on one and the other kernel, built widths, rows that take no 16-byte loads
    (3, 20, 700), (2, 9, 768), (2, 9, 772), (3, 12, 1000),      # the widest with these wavefronts, and beyond
    (3, 150, 512),                                          # several tiles a workgroup
])
def test_float(T, B, H):
    check_step(dict(T=T, B=B, D=8, H=H, L=2, P=0, V=20), 0, seed=96)


@pytest.mark.parametrize("B,H", [(8, 32), (40, 512), (20, 700), (150, 512)])
def test_float_backward_passes_on_one_forward_pass(B, H):
    # the first finds its exchange copies marked by the forward pass (one tile a workgroup), later ones and captured ones mark them
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dims = dict(T=5, B=B, D=8, H=H, L=2, P=0, V=20)
    print(f"case dims={dims}", flush=True)
    lrn = Learner(mode=0, **dims)
    g = torch.Generator(device="cuda").manual_seed(5)
    lrn.theta.copy_(torch.empty(lrn.n, device="cuda").uniform_(-0.1, 0.1, generator=g))
    lrn.x.copy_(torch.randn(lrn.x.shape, device="cuda", generator=g))
    lrn.labels.copy_(torch.randint(0, dims["V"], lrn.labels.shape, device="cuda", generator=g))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        lrn.calgrad(s)
        want = lrn.grad.clone()
        assert torch.isfinite(want).all() and want.abs().max() > 0
        backward = lambda: bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad, s)   # noqa: E731
        soft = bl.blstm_param_offset(lrn.ctx, 0, 0, bl.BLSTM_WS)[0]   # (its gradient is not this call's)
        for _ in range(2):
            lrn.grad[:soft].zero_(); backward()
            assert torch.equal(lrn.grad[:soft], want[:soft])
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            backward()
        for _ in range(3):
            lrn.grad[:soft].zero_(); graph.replay()
            s.synchronize()
            assert torch.equal(lrn.grad[:soft], want[:soft])
        lrn.check_status(s)
    lrn.close()
