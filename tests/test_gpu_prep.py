"""The launch a pass starts with (csrc/lp_conv.hip: prep_kernel): more clears and filter re-layouts than one launch holds, about
as many and few, filters of one and several 64 x 64 tiles, both storage types.  The whole step against the oracle at the
tolerance of tests/gpu_common.py: a gradient that was not cleared or a filter that was not re-laid out would be far off."""
import pytest

from tests.gpu_common import compare_step, say
from workloads import configs as cfg
from workloads.configs import Block

pytestmark = pytest.mark.gpu

PREP, MOST = 0, 96


def net_of(K, width, dtype):
    net = cfg._assemble("prep", [[Block("basic", width, width, width, 1, False)] for _ in range(K)], 3, 4, 4, 3, 1, width, 5, seed=59)
    net.dtype = dtype
    return net


@pytest.mark.parametrize("K,width,dtype", [(32, 24, "f32"), (19, 24, "f32"), (20, 24, "bf16"), (2, 72, "f32"), (1, 136, "bf16")])
def test_first_launch(K, width, dtype):
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    say("case prep", K, width, dtype)
    net = net_of(K, width, dtype)
    compare_step(net, lanes=[0] * K)
    params, _, labels, xs, lams = seeded_step_inputs(net)

    def grads(whole):
        ls = LocalStep(net)
        try:
            ls.set_stream_lanes([0] * K)
            for k in range(K):
                ls.set_params(k, params[k])
                ls.set_x(k, xs[k])
            ls.set_lams(lams)
            ls.set_labels(labels)
            for t in ls.dparams:
                t.fill_(7.0)
            B.lp_profile_enable(ls.net, 2)
            if whole:
                ls.local_step(net.rho, 1.0)
            else:
                ls.module_forward()
                ls.local_loss_grad(net.rho, 1.0)
                ls.module_backward()
            torch.cuda.synchronize()
            n = [r["nprob"] for r in B.lp_profile_fetch(ls.net) if r["kind"] == PREP]
            B.lp_profile_enable(ls.net, 0)
            return [t.clone() for t in ls.dparams], n
        finally:
            ls.close()

    one, n = grads(True)
    two, _ = grads(False)
    say("    problems of the first launches:", n)
    total = sum(n)
    assert n == [MOST] * (total // MOST) + ([total % MOST] if total % MOST else []), n
    for a, b in zip(one, two):                       # the same kernels on the same inputs, sums of up to 48 pixels in another order
        assert torch.isfinite(a).all()
        assert float((a - b).norm()) <= 1e-4 * float(b.norm())
