"""The folded kernels of the narrow networks (16 / 32 / 64 channels, csrc/lp_fconv.hip and lp_fwgrad.hip) and the small tiles
of the wide layers (csrc/lp_sconv.hip) at the sizes where their tiles, windows and dispatch rules change.

Every unit of a step is checked on its own against the oracle's float64 primitives, at the fixed tolerance of
tests/gpu_unitwise.py, and the launch records say that the path a case is about is the one that ran."""
import pytest

from tests.gpu_common import say
from tests.gpu_unitwise import check_units, seeded_step_inputs
from workloads import configs as cfg
from workloads.configs import Block

pytestmark = pytest.mark.gpu

FOLDED, FOLDED_WGRAD, CONV, SMALL_TILES = 17, 18, 2, 24


def narrow_net(batch, side, widths=(16, 32, 64), dtype="f32", c_img=3, split=None, stride=2, flags=False):
    """A block per width and one more of the last: two modules, or the given split."""
    blocks, cin = [], widths[0]
    for i, c in enumerate(widths):
        s = stride if i else 1
        blocks.append(Block("basic", cin, c, c, s, proj=(s != 1 or cin != c)))
        cin = c
    blocks.append(Block("basic", cin, cin, cin, 1, False))
    if flags:                                      # ReLU behind the sum, and a projection without a batch norm
        blocks[0].post_relu, blocks[1].post_relu, blocks[1].proj_bn = True, True, False
    net = cfg._assemble("narrow", cfg._split(blocks, split or [1, len(blocks) - 1]), batch, side[0], side[1], c_img, 1, widths[0], 5, seed=41)
    net.dtype = dtype
    return net


def wide_net(batch, side, widths, kind="basic"):
    a, b = widths
    w = (lambda c: c // 4) if kind == "bottleneck" else (lambda c: c)
    blocks = [Block(kind, a, a, w(a), 1, False), Block(kind, a, b, w(b), 2, True), Block(kind, b, b, w(b), 1, False)]
    net = cfg._assemble("wide", [blocks[:1], blocks[1:]], batch, side[0], side[1], 3, 1, a, 7, seed=43)
    net.dtype = "bf16"
    return net


def launches(net):
    """(kind, tile variant) of the launches of one local step."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        B.lp_profile_enable(ls.net, 2)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        recs = B.lp_profile_fetch(ls.net)
        B.lp_profile_enable(ls.net, 0)
    finally:
        ls.close()
    return {(r["kind"], r["cfg"]) for r in recs}


NARROW = [
    # one sample, images down to 2 x 2; one sample of the ordinary size
    dict(batch=1, side=(8, 8)), dict(batch=1, side=(32, 32)),
    # rows that are no power of two, last tiles of fewer rows, a stage without stride, images of one and two channels
    dict(batch=5, side=(12, 20)), dict(batch=3, side=(7, 9), stride=1), dict(batch=2, side=(12, 4), c_img=1),
    dict(batch=2, side=(6, 14), c_img=2, widths=(64, 16)), dict(batch=3, side=(5, 5), widths=(32, 64), stride=1),
    # the widest row a tile holds
    dict(batch=2, side=(8, 64)),
    # deep enough for the ordered tiles at any mini-batch (four blocks in a module); two images per tile with an odd rest
    dict(batch=3, side=(32, 32), split=[4]), dict(batch=33, side=(32, 32)),
    # ReLU behind the sum, bare projection
    dict(batch=3, side=(16, 16), flags=True), dict(batch=32, side=(16, 16), flags=True),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", NARROW, ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", ""))
def test_narrow_units(case, dtype):
    say("case narrow", case, dtype)
    net = narrow_net(dtype=dtype, **case)
    check_units(net, note=f" {case}")
    kinds = {k for k, _ in launches(net)}
    assert FOLDED in kinds and FOLDED_WGRAD in kinds, kinds


def test_narrow_separate_calls():
    """The single entry points run the folded passes too, each from what the one before has left in the workspace."""
    say("case narrow, separate calls")
    check_units(narrow_net(batch=3, side=(12, 20), dtype="bf16"), fused=False)


@pytest.mark.parametrize("case", [dict(batch=2, side=(4, 66), widths=(16, 32)), dict(batch=3, side=(8, 8), widths=(16, 48))],
                         ids=["rows_of_66_pixels", "48_channels"])
def test_narrow_refused(case):
    """What the folded kernels do not take goes through the general ones, whole network by whole network."""
    say("case narrow refused", case)
    net = narrow_net(dtype="bf16", **case)
    check_units(net, note=f" {case}")
    kinds = {k for k, _ in launches(net)}
    assert FOLDED not in kinds and CONV in kinds, kinds


@pytest.mark.parametrize("batch,side,dtype", [(3, (12, 20), "f32"), (2, (12, 4), "f32"), (3, (12, 20), "bf16"), (33, (16, 16), "bf16")])
def test_narrow_equals_separate_passes(batch, side, dtype):
    """The folded passes against the separate ones (the fixed-order mode runs those) on the same network: in fp32 every
    tensor agrees to 1e-4 of its largest value, which is what two orders of the same fp32 sums give; in bf16 the forward
    pass and the losses' adjoints to 2e-2 (the backward pass of a bf16 network amplifies single roundings)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.helpers import rel_err
    net = narrow_net(batch=batch, side=side, dtype=dtype)
    say("case narrow against separate passes", batch, side, dtype)
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        got = []
        for fixed in (0, 1):
            B.lp_net_set_deterministic(ls.net, fixed)
            ls.ws.zero_()
            ls.local_step(net.rho, 1.0)
            torch.cuda.synchronize()
            out = {f"y{k}": ls.y[k].clone() for k in range(net.K - 1)}
            out.update({f"dy{k}": ls.dy[k].clone() for k in range(net.K - 1)})
            out.update(logits=ls.logits.clone(), dlogits=ls.dlogits.clone())
            if dtype == "f32":
                out.update({f"dx{k}": ls.dx[k].clone() for k in range(1, net.K)})
                out.update({f"dparams{k}": ls.dparams[k].clone() for k in range(net.K)})
            got.append(out)
    finally:
        ls.close()
    tol = 1e-4 if dtype == "f32" else 2e-2
    errs = {n: rel_err(got[0][n].float().cpu().numpy(), got[1][n].float().cpu().numpy()) for n in got[0]}
    say("    worst: " + ", ".join(f"{k}={v:.1e}" for k, v in sorted(errs.items(), key=lambda kv: -kv[1])[:4]))
    assert all(v <= tol for v in errs.values()), errs


@pytest.mark.parametrize("case", [
    # one image per tile or several (8 x 8 and 4 x 4 images), an odd rest, a half last slab (160 = 2.5 slabs of 64)
    dict(batch=1, side=(8, 8), widths=(160, 320)), dict(batch=3, side=(8, 8), widths=(320, 640)), dict(batch=5, side=(16, 16), widths=(160, 320)),
    # rows that are no power of two, so that a tile ends inside an image; 1x1 layers with and without stride
    dict(batch=2, side=(12, 20), widths=(160, 320)), dict(batch=3, side=(14, 14), widths=(640, 1280), kind="bottleneck"),
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", ""))
def test_small_tiles_of_wide_layers(case):
    say("case small tiles", case)
    net = wide_net(**case)
    check_units(net, note=f" {case}")
    assert (CONV, SMALL_TILES) in launches(net)


@pytest.mark.parametrize("batch,classes,width,tiled", [
    # the last group of samples, classes and channels not full; more samples than a chunk of the filter gradient holds
    (13, 1003, 2040, (True, True)), (150, 509, 648, (True, True)), (9, 2047, 1288, (True, True)),
    # one of the two kernels tiled
    (3, 1001, 2048, (False, True)), (300, 101, 632, (True, False)),
    (150, 100, 640, (False, False))])
def test_linear_layer_kernels(batch, classes, width, tiled):
    from paper_2112_05387_amd import binding as B
    say("case linear layer", batch, classes, width)
    assert B.lp_debug_linear_kernels(batch, classes, width) == tiled
    net = cfg._assemble("linear", [[Block("bottleneck", width, width, 8, 1, False)]], batch, 2, 2, width, 0, 0, classes, seed=47)
    check_units(net)
