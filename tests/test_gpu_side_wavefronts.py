"""Recurrences whose workgroups have wavefronts of their own for what is not the exchange, four frames ahead: few frames, widths and
batches at the edges of slices, tiles and built widths, z written by the recurrence, exchange copies marked by it."""
import pytest

from test_gpu_parity import check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,H", [
    (1, 1, 8), (2, 16, 8), (3, 17, 24), (5, 50, 320),       # H below a slice, one frame, every remainder of four frames
    (4, 64, 512), (6, 49, 392), (7, 128, 256), (5, 200, 128), (5, 64, 128), (6, 500, 64), (3, 120, 72), (4, 90, 64),   # eight groups and more, through the L2; built widths
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


@pytest.mark.parametrize("mode,B,H", [(0, 8, 32), (0, 40, 512), (0, 20, 700), (0, 150, 512), (1, 8, 512), (1, 50, 320), (1, 200, 512), (1, 130, 544)])
def test_backward_passes_that_find_another_ones_exchange_copies(mode, B, H):
    # dE/da's copies are marked by the forward pass (where its kernels do), by later backward passes, by captured ones, and by those outside of a graph
    # behind a replay of one.  Another dz each time: what an earlier pass has left there gives another gradient.
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dims = dict(T=5, B=B, D=8, H=H, L=2, P=0, V=20)
    print(f"case mode={mode} dims={dims}", flush=True)
    lrn = Learner(mode=mode, **dims)
    g = torch.Generator(device="cuda").manual_seed(5)
    lrn.theta.copy_(torch.empty(lrn.n, device="cuda").uniform_(-0.1, 0.1, generator=g))
    if mode == 1:
        bl.blstm_shadow_refresh(lrn.theta, lrn.shadow, lrn.n)
    lrn.weights_changed()
    lrn.x.copy_(torch.randn(lrn.x.shape, device="cuda", generator=g))
    lrn.labels.copy_(torch.randint(0, dims["V"], lrn.labels.shape, device="cuda", generator=g))
    soft = bl.blstm_param_offset(lrn.ctx, 0, 0, bl.BLSTM_WS)[0]   # (its gradient is not this call's)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        lrn.calgrad(s)
        dzs = [torch.randn(lrn.dz.shape, device="cuda", generator=g).to(lrn.dz.dtype) for _ in range(4)]

        def backward(k):
            lrn.dz.copy_(dzs[k]); lrn.grad.zero_()
            bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad, s)
            s.synchronize()
            return lrn.grad[:soft].clone()

        want = []
        for k in range(4):
            lrn.forward(s)
            want.append(backward(k))
        assert all(torch.isfinite(w).all() and w.abs().max() > 0 for w in want) and not torch.equal(want[0], want[1])
        for k in (1, 2, 0):                                  # on one forward pass
            assert torch.equal(backward(k), want[k])
        lrn.forward(s)
        s.synchronize()
        alone, both = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(alone, stream=s):
            bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad, s)
        with torch.cuda.graph(both, stream=s):
            lrn.forward(s)
            bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad, s)
        for graph in (alone, both):
            for k in (3, 1, 2):
                lrn.forward(s)
                lrn.dz.copy_(dzs[k]); lrn.grad.zero_(); graph.replay()
                s.synchronize()
                assert torch.equal(lrn.grad[:soft], want[k])
                assert torch.equal(backward((k + 1) % 4), want[(k + 1) % 4])   # (behind the replay, which the library does not see)
        lrn.check_status(s)
    lrn.close()
