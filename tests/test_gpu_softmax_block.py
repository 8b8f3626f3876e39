"""The softmax block's two entry points: the order of the logits' sums, and that both give the same bits."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["softmax_xent_fwd_bwd", "softmax_xent_fwd_bwd_noalloc"])
@pytest.mark.parametrize("mode,slab", [(1, 64), (0, 32)])
@pytest.mark.parametrize("slabs,V", [(8, 500), (16, 500), (32, 130)])
def test_a_logit_is_summed_in_chains_of_at_least_eight_slabs(entry, mode, slab, slabs, V):
    # 2^24 in slab 3, 1 in slab 5 for the odd classes only, -2^24 in slab 7: summed in one chain the 1 is lost
    # (2^24 + 1 rounds to 2^24) and all logits are 0; with a part boundary in between (four slabs a part) it is not, and
    # the odd classes stand out
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    Z = slabs * slab
    lrn = Learner(mode=mode, T=3, B=28, D=8, H=8, L=1, P=Z, V=V, defer_softmax_wgrad=False)
    try:
        off, n = bl.blstm_param_offset(lrn.ctx, 0, 0, bl.BLSTM_WS)
        w = lrn.theta_fwd[off:off + n].view(V, Z)
        for k, zk, wk in ((3 * slab, 4096.0, 4096.0), (5 * slab, 1.0, 0.0), (7 * slab, -4096.0, 4096.0)):
            lrn.z[:, :, k] = zk
            w[:, k] = wk
        w[1::2, 5 * slab] = 1.0
        getattr(bl, entry)(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
        assert abs(lrn.loss_value() - math.log(V)) <= 1e-5 * math.log(V)
    finally:
        lrn.close()


@pytest.mark.parametrize("dims,mode", [
    (dict(T=21, B=16, D=8, H=8, L=1, P=512, V=30000), 1),   # little room behind the logits for the parts of dz
    (dict(T=21, B=16, D=8, H=8, L=1, P=1024, V=29000), 1),
    (dict(T=4, B=21, D=8, H=8, L=1, P=1024, V=500), 1),     # logits split, in a model that splits nothing else
    (dict(T=21, B=80, D=8, H=8, L=1, P=64, V=8103), 1),     # the array holds the rows of the logits unpadded only
    (dict(T=21, B=80, D=8, H=8, L=1, P=64, V=4051), 0),
    # models run as their padded twin
    (dict(T=21, B=16, D=8, H=32, L=1, P=301, V=9001), 1),
    (dict(T=21, B=16, D=8, H=32, L=1, P=1021, V=2500), 1),  # the twin's z is a whole number of 256-wide tiles
    (dict(T=5, B=40, D=8, H=101, L=1, P=0, V=900), 1),      # z in two pieces
    (dict(T=5, B=40, D=8, H=508, L=1, P=0, V=900), 1),
    (dict(T=21, B=30, D=8, H=62, L=1, P=67, V=9001), 0),
    (dict(T=21, B=30, D=8, H=301, L=1, P=0, V=3001), 0),
])
def test_both_entry_points_give_the_same_bits(dims, mode):
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    lrn = Learner(mode=mode, defer_softmax_wgrad=False, **dims)
    try:
        g = torch.Generator(device="cuda").manual_seed(4962)
        lrn.theta_fwd.copy_(0.1 * torch.randn(lrn.n, device="cuda", generator=g))
        lrn.z.copy_(torch.randn(lrn.z.shape, device="cuda", generator=g))
        lrn.labels.copy_(torch.randint(0, dims["V"], lrn.labels.shape, device="cuda", generator=g))
        out = []
        for entry in (bl.softmax_xent_fwd_bwd, bl.softmax_xent_fwd_bwd_noalloc):
            for t in (lrn.loss, lrn.dz, lrn.grad):
                t.fill_(-1.0)
            entry(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
            out.append([t.cpu().clone() for t in (lrn.loss, lrn.dz, lrn.grad)])
        for name, a, b in zip(("loss", "dz", "grad"), *out):
            assert torch.equal(a, b), (name, float((a.float() - b.float()).abs().max()), float(a.float().abs().max()))
        check_results(lrn, dims, mode)
    finally:
        lrn.close()


@pytest.mark.parametrize("B,V", [(1001, 13001), (780, 13001)])
def test_dz_on_256x256_tiles_of_many_frames(B, V):
    # 83 of these tiles in three parts, the last row tile and the last slab partial, and 64 in four
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dims = dict(T=21, B=B, D=8, H=8, L=1, P=256, V=V)
    lrn = Learner(mode=1, defer_softmax_wgrad=False, **dims)
    try:
        g = torch.Generator(device="cuda").manual_seed(4963)
        lrn.theta_fwd.copy_(0.1 * torch.randn(lrn.n, device="cuda", generator=g))
        lrn.z.copy_(torch.randn(lrn.z.shape, device="cuda", generator=g))
        lrn.labels.copy_(torch.randint(0, V, lrn.labels.shape, device="cuda", generator=g))
        bl.softmax_xent_fwd_bwd(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
        check_results(lrn, dims, 1)
    finally:
        lrn.close()


def check_results(lrn, dims, mode):
    # the softmax block's results
    import torch
    from paper_1904_04956_amd import binding as bl
    off, n = bl.blstm_param_offset(lrn.ctx, 0, 0, bl.BLSTM_WS)
    w = lrn.theta_fwd[off:off + n].double().view(dims["V"], -1).requires_grad_()
    b = lrn.theta_fwd[off + n:].double().requires_grad_()
    z = lrn.z.double().view(-1, lrn.zdim).requires_grad_()
    loss = torch.nn.functional.cross_entropy(z @ w.t() + b, lrn.labels.view(-1).long())
    loss.backward()
    loss = loss.detach()
    tol = 2e-2 if mode == 1 else 1e-4
    assert abs(lrn.loss_value() - float(loss)) <= tol * float(loss)
    for got, ref in ((lrn.dz, z.grad), (lrn.grad[off:off + n], w.grad), (lrn.grad[off + n:], b.grad)):
        assert float((got.double().view(-1) - ref.reshape(-1)).abs().max()) <= tol * float(ref.abs().max())
