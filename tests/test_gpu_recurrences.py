"""The persistent bf16 recurrences: results that must not depend on which unit, which way of exchange or which launch of a
pass they come from.  Bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


def learner(dims, seed, **options):
    """A learner with weights and a batch drawn on the device from the seed."""
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    print(f"case dims={dims} seed={seed} {options}", flush=True)
    lrn = Learner(mode=1, **dims, **options)
    g = torch.Generator(device="cuda").manual_seed(seed)
    lrn.theta.copy_(torch.empty(lrn.n, device="cuda").uniform_(-0.1, 0.1, generator=g))
    bl.blstm_shadow_refresh(lrn.theta, lrn.shadow, lrn.n)
    lrn.weights_changed()
    lrn.x.copy_(torch.randn(lrn.x.shape, device="cuda", generator=g) * 2)
    lrn.labels.copy_(torch.randint(0, dims["V"], lrn.labels.shape, device="cuda", generator=g))
    return lrn


@pytest.mark.parametrize("T,B,H", [
    (300, 1000, 128), (600, 500, 256), (900, 300, 384), (800, 256, 512),    # one 16-row tile a workgroup, slices of 64 units
    (2000, 100, 512), (100, 2048, 64),                                      # of 32, and two workgroups a CU
    (300, 600, 512), (2000, 64, 512), (200, 200, 1024),                     # several tiles, few sequences, wide layers
])
def test_units_with_the_same_weights_give_the_same_bits(T, B, H):
    # Every unit's rows of W_x and b are the same and U_h is zero (wavefronts contract it in orders of their own): so are c and h, in every
    # frame of 2e5 rows or so.  (One rounding of c shows in h's bf16 once in some 1e5 cells.)
    import torch
    from paper_1904_04956_amd import binding as bl
    lrn = learner(dict(T=T, B=B, D=8, H=H, L=1, P=0, V=8), 7)
    for d in range(2):
        for which in (bl.BLSTM_WX, bl.BLSTM_UH, bl.BLSTM_B):
            off, n = bl.blstm_param_offset(lrn.ctx, 0, d, which)
            w = lrn.theta[off:off + n].view(4, H, -1)
            w.copy_(w[:, :1].clone().expand_as(w) * {bl.BLSTM_WX: 3.0, bl.BLSTM_UH: 0.0, bl.BLSTM_B: 1.0}[which])
    bl.blstm_shadow_refresh(lrn.theta, lrn.shadow, lrn.n)
    lrn.weights_changed()
    lrn.forward()
    lrn.check_status()
    z = lrn.z.view(T * B, 2, H)
    assert torch.isfinite(z.float()).all()
    differ = (z != z[:, :, :1]).sum(dim=(0, 1))
    others = torch.nonzero(differ).flatten().tolist()
    assert not others, f"units that differ from the first: {others[:8]}"
    lrn.close()


@pytest.mark.parametrize("B,H", [(256, 1024), (130, 544), (16, 512), (128, 512), (600, 512), (1300, 136)])
def test_a_captured_backward_pass_replayed_twice_on_one_forward_pass(B, H):
    # other gradients of z each time, as launched calls give them
    import torch
    from paper_1904_04956_amd import binding as bl
    lrn = learner(dict(T=5, B=B, D=8, H=H, L=2, P=0, V=20), 11)
    s = torch.cuda.Stream()
    backward = lambda stream: bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad, stream)   # noqa: E731
    with torch.cuda.stream(s):
        lrn.calgrad(s)
        lrn.check_status(s)
        g = torch.Generator(device="cuda").manual_seed(3)
        dzs = [torch.randn(lrn.dz.shape, device="cuda", generator=g).to(lrn.dz.dtype) for _ in range(3)]
        expected = []
        for dz in dzs:
            lrn.forward(s); lrn.dz.copy_(dz); lrn.grad.zero_(); backward(s)
            s.synchronize()
            expected.append(lrn.grad.clone())
        lrn.forward(s)
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            backward(s)
        for dz, want in zip(dzs, expected):
            lrn.dz.copy_(dz); lrn.grad.zero_()
            graph.replay()
            s.synchronize()
            assert torch.equal(lrn.grad, want)
        lrn.check_status(s)
    lrn.close()


@pytest.mark.parametrize("B,H", [
    (500, 128), (250, 256), (500, 256), (1000, 128),        # one 16-row tile a workgroup
    (700, 136), (400, 264), (1500, 128), (2600, 40), (2049, 24), (4130, 32),        # ... and several workgroups a CU
    (272, 512), (600, 512), (3340, 512), (2100, 256), (3000, 320), (3000, 128),   # several tiles, at 272 a group of a neighbour's too
    (64, 512), (49, 392), (64, 128), (180, 72), (250, 64), (500, 24),   # few sequences
])
def test_exchange_through_the_memory_side_gives_the_same_bits(B, H):
    # groups on one XCD exchange through its L2 where the kernels ask; told that none is, they write through
    import torch
    from paper_1904_04956_amd import binding as bl
    lrn = learner(dict(T=6, B=B, D=8, H=H, L=2, P=0, V=20), 13)
    results = []
    for no_xcd in (0, 1, 0):
        bl.blstm_set_option(lrn.ctx, bl.BLSTM_OPT_TEST_NO_XCD, no_xcd)
        for _ in range(2):
            lrn.grad.zero_()
            lrn.calgrad()
        lrn.check_status()
        results.append((lrn.loss.clone(), lrn.z.clone(), lrn.grad.clone()))
    assert torch.isfinite(results[0][2]).all()
    for r in results[1:]:
        assert all(torch.equal(a, b) for a, b in zip(r, results[0]))
    lrn.close()


@pytest.mark.parametrize("B,H", [(200, 1024), (130, 544), (1500, 128), (400, 264), (60, 512), (3340, 512)])
def test_abandoned_waits_of_the_other_kernels(B, H):
    # raised from the host, as in test_gpu_parity.py: the forms of the wide layers that look ahead, several workgroups a CU, carried state in memory
    import torch
    from paper_1904_04956_amd import binding as bl
    lrn = learner(dict(T=6, B=B, D=8, H=H, L=2, P=0, V=20), 17)
    lrn.calgrad(); lrn.check_status()
    clean = lrn.grad.clone()
    assert torch.isfinite(clean).all()
    bl.blstm_set_option(lrn.ctx, bl.BLSTM_OPT_TEST_ABORT, 1)
    lrn.calgrad()
    with pytest.raises(bl.BlstmError) as e:
        lrn.check_status()
    assert e.value.code == -5 and "abandoned" in str(e.value)
    assert torch.isnan(lrn.loss).all() and torch.isnan(lrn.z).any() and torch.isnan(lrn.grad).any()
    lrn.calgrad(); lrn.check_status()
    assert torch.equal(lrn.grad, clean)
    lrn.close()


@pytest.mark.parametrize("T,B,H", [
    (2, 700, 256), (5, 520, 320), (3, 449, 384),     # two tiles a workgroup: the look is timed
    (4, 1300, 256),                                  # two in some, three in others
])
def test_backward_looks_behind_a_pause(T, B, H):
    from test_gpu_parity import check_step
    check_step(dict(T=T, B=B, D=8, H=H, L=2, P=0, V=20), 1, seed=98, theta_scale=2.0)
