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


@pytest.mark.parametrize("dims,mode", [
    (dict(T=5, B=40, D=30, H=101, L=2, P=40, V=90), 1),
    (dict(T=5, B=40, D=32, H=125, L=1, P=0, V=90), 1),      # the twin has a width with kernels of its own
    (dict(T=21, B=60, D=33, H=66, L=2, P=67, V=9001), 0),
])
@pytest.mark.parametrize("path", [0, 1])
def test_infinite_features_saturate_the_gates(dims, mode, path):
    # +-inf times a weight is +-inf: the gates saturate and z is finite, in the frames before and behind it too
    from oracle import blstm_oracle as orc
    from paper_1904_04956_amd.harness import Learner
    dm, theta, x, labels = make_problem(dims, mode, 91, 2.0)
    x[2, 3, 7] = np.inf; x[1, 4, 0] = -np.inf
    lrn = Learner(mode=mode, recurrent_path=path, **dims)
    try:
        lrn.set_theta(theta); lrn.set_batch(x, labels)
        lrn.forward(); lrn.check_status()
        z = lrn.z_numpy()
    finally:
        lrn.close()
    with np.errstate(all="ignore"):
        ref, _ = orc.blstm_forward(dm, theta.astype(np.float64), x)
    assert np.isfinite(ref).all()
    assert int(np.sum(~np.isfinite(z))) == 0
    assert np.abs(z - ref).max() <= (2e-2 if mode == 1 else 1e-4) * np.abs(ref).max()


@pytest.mark.parametrize("D", [7, 31, 33])                 # rows of W_x that start at any even address, one shorter than a word
def test_feature_widths_the_twin_leaves_as_they_are(D):
    check_step(dict(T=4, B=9, D=D, H=101, L=1, P=0, V=40), 1, seed=92, theta_scale=2.0)


@pytest.mark.parametrize("dims,mode", [(TWIN, 1), (dict(T=21, B=60, D=33, H=66, L=2, P=67, V=9001), 0)])
def test_one_launch_per_frame(dims, mode):
    check_step(dims, mode, seed=94, theta_scale=2.0, recurrent_path=1)


@pytest.mark.parametrize("dims,mode", [(TWIN, 1), (dict(T=21, B=60, D=33, H=66, L=2, P=67, V=9001), 0)])
def test_abandoned_wait_is_reported_and_recovered_from(dims, mode):
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dm, theta, x, labels = make_problem(dims, mode, 95, 2.0)
    lrn = Learner(mode=mode, **dims)
    try:
        lrn.set_theta(theta); lrn.set_batch(x, labels)
        lrn.calgrad(); lrn.check_status()
        clean = (lrn.loss_value(), lrn.grad_numpy().copy())
        bl.blstm_set_option(lrn.ctx, bl.BLSTM_OPT_TEST_ABORT, 1)
        lrn.calgrad()
        code, text = 0, ""
        try:                                               # (a kept exception keeps this frame, and with it the learner's device memory, until some later collection)
            lrn.check_status()
        except bl.BlstmError as e:
            code, text = e.code, str(e)
        assert code == -5 and "abandoned" in text
        assert np.isnan(lrn.loss_value()) and np.isnan(lrn.grad_numpy()).any()
        lrn.calgrad(); lrn.check_status()
        assert lrn.loss_value() == clean[0] and np.array_equal(lrn.grad_numpy(), clean[1])
    finally:
        lrn.close()


def test_noalloc_call_between_the_passes_changes_nothing_else():
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dm, theta, x, labels = make_problem(TWIN, 1, 96, 2.0)
    lrn = Learner(mode=1, defer_softmax_wgrad=False, **TWIN)
    try:
        lrn.set_theta(theta); lrn.set_batch(x, labels)
        lrn.calgrad()
        ref = lrn.grad.clone()
        loss, dz, grad = torch.zeros_like(lrn.loss), torch.zeros_like(lrn.dz), torch.zeros_like(lrn.grad)
        other = (lrn.labels + 1) % TWIN["V"]
        for when in range(2):                              # before the softmax block, and behind it
            lrn.grad.zero_()
            lrn.forward()
            if when == 0:
                bl.softmax_xent_fwd_bwd_noalloc(lrn.ctx, lrn.theta_fwd, lrn.z, other, loss, dz, grad)
            bl.softmax_xent_fwd_bwd(lrn.ctx, lrn.theta_fwd, lrn.z, lrn.labels, lrn.loss, lrn.dz, lrn.grad)
            if when == 1:
                bl.softmax_xent_fwd_bwd_noalloc(lrn.ctx, lrn.theta_fwd, lrn.z, other, loss, dz, grad)
            bl.blstm_backward(lrn.ctx, lrn.theta_fwd, lrn.x, lrn.dz, lrn.grad)
            assert torch.equal(lrn.grad, ref)
    finally:
        lrn.close()


@pytest.mark.parametrize("defer", [False, True])
def test_softmax_weights_need_no_report(defer):
    # kept copies are promised to blstm_forward and blstm_backward only: softmax_xent_fwd_bwd reads the weights as they are
    import torch
    from paper_1904_04956_amd import binding as bl
    from paper_1904_04956_amd.harness import Learner
    dm, theta, x, labels = make_problem(TWIN, 1, 97, 2.0)
    a, b = (Learner(mode=1, defer_softmax_wgrad=defer, keep_weight_copies=keep, **TWIN) for keep in (True, False))
    try:
        for l in (a, b):
            l.set_theta(theta); l.set_batch(x, labels)
            l.calgrad()
            off, n = bl.blstm_param_offset(l.ctx, 0, 0, bl.BLSTM_WS)
            l.theta_fwd[off:off + n] *= 0.5
            l.calgrad()                                    # (nothing reported; only the softmax layer has changed)
        assert torch.equal(a.loss, b.loss) and torch.equal(a.dz, b.dz) and torch.equal(a.grad, b.grad)
    finally:
        a.close(); b.close()
