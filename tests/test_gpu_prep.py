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


@pytest.mark.parametrize("batch,side,width,classes,dtype,one", [
    # one pixel, one class; fewer channels than a wave has lanes, a second round of classes; more channels than lanes
    (1, (1, 1), 16, 1, "f32", True), (3, (4, 4), 16, 23, "f32", True), (5, (3, 3), 72, 7, "bf16", True), (2, (8, 4), 200, 81, "f32", True),
    # a round of classes and one more
    (4, (4, 4), 64, 32, "f32", True), (4, (4, 4), 64, 33, "bf16", True),
    # the largest sample (32 KB) and the most weights (16384) of the rule, and one more of each
    (2, (16, 8), 64, 256, "f32", True), (2, (17, 8), 64, 10, "f32", False), (2, (4, 4), 64, 257, "bf16", False)])
def test_head_with_loss(batch, side, width, classes, dtype, one):
    """Pooling, linear layer and cross-entropy of a small head in one launch of the whole step: the logits, their gradients and the losses of
    the single entry points, which launch them one after the other; every step clears the losses it adds to."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    say("case head with loss", batch, side, width, classes, dtype)
    net = cfg._assemble("head", [[Block("basic", width, width, width, 1, False)] for _ in range(2)], batch, side[0], side[1], 3, 1, width, classes, seed=61)
    net.dtype = dtype
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(2):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        ls.module_forward()
        ls.local_loss_grad(net.rho, 1.0)
        want = [t.clone() for t in (ls.logits, ls.dlogits, ls.loss, ls.r2)]
        for t in (ls.logits, ls.dlogits, ls.loss, ls.r2):
            t.fill_(7.0)
        B.lp_profile_enable(ls.net, 2)
        for _ in range(2):
            ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        kinds = {r["kind"] for r in B.lp_profile_fetch(ls.net)}
        B.lp_profile_enable(ls.net, 0)
        assert (13 in kinds) == (not one), kinds
        for a, b in zip((ls.logits, ls.dlogits), want):
            assert torch.equal(a, b) if net.dtype == "f32" else float((a - b).abs().max()) <= 1e-6 * float(b.abs().max() + 1.0)
        for a, b in zip((ls.loss, ls.r2), want[2:]):      # atomics of up to 50 workgroups in another order
            assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max() + 1.0)
    finally:
        ls.close()


@pytest.mark.parametrize("modules,lanes", [(1, None), (2, None), (2, [0, 1]), (3, [0, 1, 0])])
def test_last_pass_evaluates_a_loss_only_in_company(modules, lanes):
    """The last module's last pass has no loss (its head has it): in a lane of its own it is the plain pass, with others of its lane it
    shares their launch, and its record counts the tensors that it reads and writes."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    say("case last pass", modules, lanes)
    batch, width = 2, 16
    net = cfg._assemble("last", [[Block("basic", width, width, width, 1, False)] for _ in range(modules)], batch, 8, 8, 3, 1, width, 5, seed=79)
    net.dtype = "f32"
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(modules):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        ls.set_stream_lanes(lanes)
        B.lp_profile_enable(ls.net, 2)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        recs = [(r["cfg"], r["nprob"], r["bytes"]) for r in B.lp_profile_fetch(ls.net) if r["kind"] == 3]
        B.lp_profile_enable(ls.net, 0)
    finally:
        ls.close()
    tensor = batch * 8 * 8 * width * 4
    plain, loss = 3 * tensor, 6 * tensor           # y, skip, out; and x_next, lam, dy
    in_lane = [[k for k in range(modules) if (lanes or [0] * modules)[k] == l] for l in range(2)]
    want = []
    for ks in in_lane:
        with_loss = sum(k < modules - 1 for k in ks)
        if ks:
            want.append((1 if with_loss else 0, len(ks), with_loss * loss + (len(ks) - with_loss) * plain))
    assert sorted(recs) == sorted(want), (recs, want)
