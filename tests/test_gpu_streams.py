"""Several learners at once: on streams of their own, from threads of their own, and in a captured graph."""
import threading

import numpy as np
import pytest

from test_gpu_parity import make_problem

pytestmark = pytest.mark.gpu

# recurrences of up to one workgroup per CU, of two, a twin, and float ones
MODELS = [(dict(T=6, B=64, D=24, H=512, L=2, P=0, V=300), 0), (dict(T=6, B=256, D=24, H=512, L=2, P=64, V=300), 1),
          (dict(T=6, B=1000, D=24, H=256, L=1, P=0, V=100), 1), (dict(T=6, B=40, D=30, H=101, L=2, P=37, V=90), 1)]


def _learner(i):
    from paper_1904_04956_amd.harness import Learner
    dims, mode = MODELS[i]
    dm, theta, x, labels = make_problem(dims, mode, 93 + i, 2.0)
    lrn = Learner(mode=mode, **dims)
    lrn.set_theta(theta); lrn.set_batch(x, labels)
    return lrn


def _result(lrn):
    return lrn.loss_value(), lrn.grad_numpy().copy()


@pytest.mark.parametrize("pair", [(0, 0), (0, 1), (1, 2), (2, 3)])
def test_two_learners_on_two_streams_give_what_each_gives_alone(pair):
    import torch
    learners = [_learner(i) for i in pair]
    try:
        alone = []
        for l in learners:
            l.calgrad(); l.check_status(); alone.append(_result(l))
            l.grad.zero_(); l.loss.zero_()
        torch.cuda.synchronize()
        failures = []

        def work(l):
            try:
                s = torch.cuda.Stream()
                for _ in range(8):
                    l.calgrad(s)
                s.synchronize()
                l.check_status(s)
            except Exception as e:                         # noqa: BLE001 (reported by the main thread)
                failures.append(e)
        threads = [threading.Thread(target=work, args=(l,)) for l in learners]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not failures, failures
        for l, (loss, grad) in zip(learners, alone):
            assert l.loss_value() == loss and np.array_equal(l.grad_numpy(), grad)
    finally:
        for l in learners:
            l.close()


@pytest.mark.parametrize("i", range(len(MODELS)))
def test_a_captured_step_replays_to_the_eager_result(i):
    import torch
    l = _learner(i)
    try:
        s = torch.cuda.Stream()
        for _ in range(2):
            l.calgrad(s)
        s.synchronize()
        loss, grad = _result(l)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            l.calgrad(s)
        for _ in range(3):
            l.grad.zero_(); l.loss.zero_()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert l.loss_value() == loss and np.array_equal(l.grad_numpy(), grad)
            l.calgrad(); l.check_status()                  # eager work in between
            assert l.loss_value() == loss and np.array_equal(l.grad_numpy(), grad)
    finally:
        l.close()
