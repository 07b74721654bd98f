"""Batch-norm apply passes whose workgroups have a slice of the channels (csrc/lp_kernels.h: bn_slice): slices of 64 and 128
channels, one and several of them, rows that do not fill a workgroup, projections and added gradients, and tensors either side of
the size from which a thread takes two trips of loads.  Units against the oracle's float64 primitives; and the slices against
whole rows, bit by bit, over an iteration that distils AuxNets from single roundings of the auxiliary variables."""
import pytest

from tests.gpu_common import compare_step, say
from tests.gpu_unitwise import check_units
from workloads import configs as cfg
from workloads.configs import Block

pytestmark = pytest.mark.gpu


def net_of(batch, side, widths, dtype, kind="basic"):
    a, b = widths
    w = (lambda c: c // 4) if kind == "bottleneck" else (lambda c: c)
    blocks = [Block(kind, a, a, w(a), 1, False), Block(kind, a, b, w(b), 2, True), Block(kind, b, b, w(b), 1, False)]
    net = cfg._assemble("slices", [blocks[:2], blocks[2:]], batch, side[0], side[1], 3, 1, a, 7, seed=61)
    net.dtype = dtype
    return net


@pytest.mark.parametrize("case", [
    dict(batch=2, side=(4, 4), widths=(128, 256), dtype="f32"), dict(batch=3, side=(6, 10), widths=(192, 384), dtype="f32"),
    dict(batch=5, side=(6, 10), widths=(128, 320), dtype="bf16"), dict(batch=2, side=(14, 6), widths=(1024, 2048), dtype="bf16", kind="bottleneck"),
    dict(batch=41, side=(40, 40), widths=(128, 256), dtype="bf16", kind="bottleneck"),       # 513 x 2048 vectors in the first block
], ids=lambda c: "-".join(str(v) for v in c.values()).replace(" ", ""))
def test_units(case):
    say("case bn slices", case)
    check_units(net_of(**case), note=f" {case}")


def test_pre_activation():
    """The identity skip's gradient added in the backward pass."""
    say("case bn slices, pre-activation")
    compare_step(cfg.with_order(net_of(3, (6, 10), (128, 192), "f32"), "pre"))


def iteration(net, whole_rows, lanes, fixed):
    """What an iteration leaves: everything but the parameter gradients, whose partial sums meet in atomics, and those."""
    import torch
    import workloads as wl
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    params, _, labels, xs, lams = seeded_step_inputs(net)
    B.lp_debug_separate_passes(whole_rows)
    try:
        ls = LocalStep(net)
    finally:
        B.lp_debug_separate_passes(False)
    try:
        if lanes is not None:
            ls.set_stream_lanes(lanes)
        B.lp_net_set_deterministic(ls.net, fixed)
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        for j in range(net.K - 1):
            ls.set_aux_params(j, wl.make_aux_params(net, j))
        ls.set_lams(lams)
        ls.set_labels(labels)
        scale = 1.0 / ls.x[1].numel()
        ls.auxnet_forward()
        ls.local_step(net.rho, scale, 0.0)
        ls.aux_variable_update(net.rho, scale, 0.1)
        ls.auxnet_distill_grad(scale)
        torch.cuda.synchronize()
        exact = {f"{n}{k}": t.clone() for n, ts in (("y", ls.y), ("dy", ls.dy), ("dx", ls.dx[1:]), ("x", ls.x[1:])) for k, t in enumerate(ts)}
        sums = {f"{n}{k}": t.clone() for n, ts in (("dparams", ls.dparams), ("daux", ls.daux_params)) for k, t in enumerate(ts)}
        return exact, sums
    finally:
        ls.close()


@pytest.mark.parametrize("case,order,lanes,fixed", [
    # several parts of the rows in a workgroup and one; row lanes that leave threads over (160: whole rows, in launches of their own)
    (dict(batch=48, side=(32, 32), widths=(160, 320), dtype="bf16"), "post", None, False),
    (dict(batch=96, side=(16, 16), widths=(192, 640), dtype="bf16"), "pre", None, False),
    (dict(batch=6, side=(14, 14), widths=(1024, 2048), dtype="bf16", kind="bottleneck"), "post", None, False),
    (dict(batch=9, side=(12, 20), widths=(192, 384), dtype="f32"), "post", None, False),
    # tensors of both kinds in one launch
    (dict(batch=5, side=(16, 16), widths=(160, 320), dtype="bf16"), "post", [0, 0], False),
    # fixed order: one part
    (dict(batch=5, side=(16, 16), widths=(256, 320), dtype="bf16"), "post", None, True),
], ids=lambda c: "-".join(str(v) for v in c.values()).replace(" ", "") if isinstance(c, dict) else str(c).replace(" ", ""))
def test_slices_have_the_bits_of_whole_rows(case, order, lanes, fixed):
    import torch
    say("case bn slices, bits of an iteration", case, order, lanes, fixed)
    net = cfg.with_order(net_of(**case), order)
    m0 = net.modules[0]
    net.aux = [cfg.AuxDesc(cin=m0.C, cout=m.C, stride=m0.H // m.H, relu=False) for m in net.modules[1:]]
    got, got_sums = iteration(net, False, lanes, fixed)
    want, want_sums = iteration(net, True, lanes, fixed)
    differ = {n: int((got[n] != want[n]).sum()) for n in got if not torch.equal(got[n], want[n])}
    say(f"    {len(got)} tensors, differing: {differ}")
    assert not differ, differ
    for n, g in got_sums.items():                  # fp32 sums of up to 2^16 products in two orders
        assert torch.isfinite(g).all() and float((g - want_sums[n]).norm()) <= 1e-5 * float(want_sums[n].norm()), n


@pytest.mark.parametrize("case,order,fixed", [
    # one row; fewer rows than a trip has; rows that end inside a trip and inside a part, several rounds of parts (256 channels and less)
    (dict(batch=1, side=(2, 2), widths=(128, 256), dtype="bf16"), "post", False), (dict(batch=3, side=(6, 10), widths=(192, 320), dtype="bf16"), "post", False),
    # the most rows that one workgroup takes, more of them beside fewer; the added gradient of an identity skip
    (dict(batch=6, side=(10, 10), widths=(128, 640), dtype="bf16"), "post", False), (dict(batch=7, side=(10, 10), widths=(192, 384), dtype="bf16"), "pre", False),
    (dict(batch=5, side=(8, 8), widths=(256, 576), dtype="bf16"), "pre", False),
    (dict(batch=7, side=(8, 8), widths=(128, 640), dtype="bf16"), "post", False), (dict(batch=8, side=(8, 8), widths=(640, 192), dtype="bf16"), "pre", False),
    # two row lanes and trips in a row, a projection's batch norm in the same launch; the fixed order takes two launches
    (dict(batch=3, side=(14, 14), widths=(1024, 2048), dtype="bf16", kind="bottleneck"), "post", False),
    (dict(batch=3, side=(6, 10), widths=(192, 320), dtype="bf16"), "post", True),
], ids=lambda c: "-".join(str(v) for v in c.values()).replace(" ", "") if isinstance(c, dict) else str(c).replace(" ", ""))
def test_few_rows_in_one_launch(case, order, fixed):
    """Reduction and apply pass of few rows in one launch: the bits of the two."""
    import torch
    from tests.test_gpu_narrow import launches
    say("case few rows", case, order, fixed)
    net = cfg.with_order(net_of(**case), order)
    assert 19 in {k for k, _ in launches(net)}
    m0 = net.modules[0]
    net.aux = [cfg.AuxDesc(cin=m0.C, cout=m.C, stride=m0.H // m.H, relu=False) for m in net.modules[1:]]
    got, got_sums = iteration(net, False, None, fixed)
    want, want_sums = iteration(net, True, None, fixed)
    differ = {n: int((got[n] != want[n]).sum()) for n in got if not torch.equal(got[n], want[n])}
    assert not differ, differ
    for n, g in got_sums.items():                  # fp32 sums of up to 2^10 products in two orders
        assert torch.isfinite(g).all() and float((g - want_sums[n]).norm()) <= 1e-5 * float(want_sums[n].norm()), n
