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
