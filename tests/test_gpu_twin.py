"""Models whose widths are no whole 16-byte words run as a zero-padded twin: what a caller may do around the plain step
must have the same effect as without one."""
import numpy as np
import pytest

from test_gpu_parity import check_step, make_problem

pytestmark = pytest.mark.gpu

TWIN = dict(T=5, B=40, D=30, H=101, L=2, P=37, V=90)       # every width misaligned
PLAIN = dict(T=5, B=40, D=32, H=104, L=2, P=40, V=90)      # none


@pytest.mark.parametrize("dims", [PLAIN, TWIN])
def test_noalloc_call_takes_over_from_a_deferred_softmax_gradient(dims):
    # the deferred call leaves W_s's slice to blstm_backward; a call that writes the slice itself ends that
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dm, theta, x, labels = make_problem(dims, 1, 90, 2.0)
    lrn = Learner(mode=1, defer_softmax_wgrad=True, **dims)
    try:
        lrn.set_theta(theta); lrn.set_batch(x, labels)
        lrn.forward()
        bl.softmax_xent_fwd_bwd(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
        other = (lrn.labels + 1) % dims["V"]
        bl.softmax_xent_fwd_bwd_noalloc(lrn.ctx, lrn.theta_fwd, lrn.z, other, lrn.loss, lrn.dz, lrn.grad)
        off, n = bl.blstm_param_offset(lrn.ctx, 0, 0, bl.BLSTM_WS)
        ws = lrn.grad[off:].clone()                        # W_s and b_s
        bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad)
        assert torch.equal(lrn.grad[off:], ws)
        bl.softmax_xent_fwd_bwd_noalloc(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
        assert not torch.equal(lrn.grad[off:], ws)
    finally:
        lrn.close()
