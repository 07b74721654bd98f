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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width,stride,bn,batch", [(16, 1, True, 3), (16, 1, False, 3), (16, 2, True, 3), (16, 2, False, 33), (32, 1, False, 3), (64, 2, True, 2)])
def test_projections_of_equal_width(width, stride, bn, batch, dtype):
    """A projection whose input and output have the same width, 1x1 filters of 16 x 16 channels among them: every unit against float64, and
    nothing written around the gradients (in the gaps between the tensors there may be zeros of the clear)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    say("case projection of equal width", width, stride, bn, batch, dtype)
    blocks = [Block("basic", width, width, width, 1, False), Block("basic", width, width, width, stride, True, proj_bn=bn),
              Block("basic", width, width, width, 1, False)]
    net = cfg._assemble("square", [blocks[:2], blocks[2:]], batch, 16, 8, 3, 1, width, 5, seed=71)
    net.dtype = dtype
    check_units(net, note=f" {width}, stride {stride}, bn {bn}")
    assert FOLDED_WGRAD in {k for k, _ in launches(net)}
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        guard, all_of = 4096, []
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
            n = ls.dparams[k].numel()
            all_of.append(torch.full((n + 2 * guard,), 7.0, device=ls.dev))
            ls.dparams[k] = all_of[k][guard:guard + n]
        ls.set_lams(lams)
        ls.set_labels(labels)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        for k in range(net.K):
            outside = torch.ones_like(all_of[k], dtype=torch.bool)
            for info in ls.tables[k]:
                o = guard + info.grad_offset // 4
                outside[o:o + int(info.numel)] = False
            v = all_of[k]
            assert bool((v[:guard] == 7.0).all()) and bool((v[-guard:] == 7.0).all()), k
            assert bool(((v == 7.0) | (v == 0.0))[outside].all()), k
    finally:
        ls.close()


@pytest.mark.parametrize("batch,side,stride", [(1, (8, 8), 2), (9, (12, 20), 2), (3, (7, 9), 1), (32, (32, 32), 2)])
def test_fp32_filter_gradients(batch, side, stride):
    """The fp32 filter gradients of every layer of a step to the precision of fp32 sums: 1e-6 (2-norm) against float64, where their chains give
    1e-7 to 4e-7; with operands cut to 16 bits it would be 2^-18 / sqrt(3) = 2e-6 or more."""
    import numpy as np
    import torch
    from oracle import lpref
    from paper_2112_05387_amd import LocalStep
    say("case fp32 filter gradients", batch, side, stride)
    net = narrow_net(batch, side, dtype="f32", stride=stride)
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net, keep_gradients=True)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        for k in range(net.K):
            grads = ls.get_grads(k)
            for u in ls.units(k):
                x, dy = ls.fetch(u.in_, (u.N, u.H, u.W, u.cin)), ls.fetch(u.dy, (u.N, u.Ho, u.Wo, u.cout))
                want = lpref.conv_wgrad(x, dy, params[k][u.t_w].shape, u.stride, u.pad)
                err = np.linalg.norm(grads[u.t_w] - want) / np.linalg.norm(want)
                say(f"  m{k} {u.cin} -> {u.cout}, {u.R}x{u.R}/{u.stride}: {err:.1e}")
                assert err < 1e-6, (k, u.cin, u.cout, err)
    finally:
        ls.close()


def middle_module(width, batch, side):
    """A module between two others, of one block of `width` channels with a bare projection: its input and the gradient of its output are the
    caller's, and so are both operands of the projection's filter gradient."""
    from paper_2112_05387_amd import LocalStep
    import workloads as wl
    blocks = lambda proj: [Block("basic", width, width, width, 1, proj, proj_bn=False)]  # noqa: E731
    net = cfg._assemble("middle", [blocks(False), blocks(True), blocks(False)], batch, side, side, 3, 1, width, 5, seed=73)
    ls = LocalStep(net, keep_gradients=True)
    ls.set_params(1, wl.make_params(net, 1))
    return ls


@pytest.mark.parametrize("width", [16, 32, 64])
def test_fp32_filter_gradients_of_one_sign(width):
    """Over many pixels whatever every product is short of adds up where the operands have one sign, and the batch norm behind the first
    convolution takes the mean of dY out, so that the large sums cancel.  Sums rounded to nearest (2-norm against float64): a chain of n terms is off by
    2^-24 sqrt(n / 6) of its random walk; 32 k-steps of a tile and 512 workgroups one after the other give 6e-7, seen are up to 5e-7.  Products cut
    at 2^-24 of the largest of eight, towards zero: 2.9e-6 with 32 channels.  (64 channels take this kernel up to 32768 pixels.)"""
    import torch
    import torch.nn.functional as F
    batch = 32 if width == 64 else 128
    say("case filter gradients of one sign", width, batch)
    from paper_2112_05387_amd import binding as B
    ls = middle_module(width, batch, 32)
    try:
        g = torch.Generator(device=ls.dev)
        g.manual_seed(5)
        ls.x[1].copy_(torch.rand(ls.x_shapes[1], generator=g, device=ls.dev))
        ls.dy[1].copy_(torch.rand(ls.x_shapes[1], generator=g, device=ls.dev))
        B.lp_profile_enable(ls.net, 2)
        ls.module_forward(mask=2)
        ls.module_backward(mask=2)
        torch.cuda.synchronize()
        kinds = {r["kind"] for r in B.lp_profile_fetch(ls.net)}
        B.lp_profile_enable(ls.net, 0)
        assert FOLDED_WGRAD in kinds, kinds
        grads = ls.get_grads(1)
        dev = lambda ref, u, c: torch.from_numpy(ls.fetch(ref, (u.N, u.H, u.W, c))).to(ls.dev)  # noqa: E731
        for u in ls.units(1):
            x, dy = dev(u.in_, u, u.cin), dev(u.gout if u.plain else u.dy, u, u.cout).reshape(-1, u.cout)
            xp = F.pad(x, (0, 0, u.pad, u.pad, u.pad, u.pad))
            want = torch.stack([dy.t().contiguous() @ xp[:, r:r + u.H, s:s + u.W].reshape(-1, u.cin) for r in range(u.R) for s in range(u.R)], 1)
            got = torch.from_numpy(grads[u.t_w]).to(ls.dev).reshape(want.shape)
            err = float((got - want).norm() / want.norm())
            say(f"  {u.R}x{u.R}: {err:.1e}")
            assert err < 1.2e-6, (width, u.R, err)
    finally:
        ls.close()


def test_infinities_in_fp32_filter_gradients():
    """An infinite element of a gradient makes its own row of a filter gradient infinite, and no other; the largest finite values multiply as
    such."""
    import numpy as np
    import torch
    say("case infinities")
    ls = middle_module(32, 2, 8)
    try:
        u = next(u for u in ls.units(1) if u.plain)
        rng = np.random.default_rng(3)
        x = rng.uniform(0.5, 1.0, ls.x_shapes[1]).astype(np.float32)
        dy = rng.uniform(0.5, 1.0, ls.x_shapes[1]).astype(np.float32)
        dy[1, 3, 4, 7], dy[0, 2, 2, 9] = np.inf, -np.inf
        x[..., 5] *= np.float32(1e-6)
        dy[1, 0, 1, 11] = np.float32(3.4e38)
        ls.x[1].copy_(torch.from_numpy(x))
        ls.dy[1].copy_(torch.from_numpy(dy))
        ls.module_forward(mask=2)
        ls.module_backward(mask=2)
        torch.cuda.synchronize()
        got = ls.get_grads(1)[u.t_w].reshape(32, 32)
        with np.errstate(invalid="ignore"):
            want = dy.reshape(-1, 32).T.astype(np.float64) @ x.reshape(-1, 32).astype(np.float64)
        assert (got[7] == np.inf).all() and (got[9] == -np.inf).all(), (got[7], got[9])
        rows = [r for r in range(32) if r not in (7, 9)]
        assert (np.abs(got[rows] - want[rows]) <= 1e-5 * np.abs(want[rows])).all()
    finally:
        ls.close()


@pytest.mark.parametrize("blocks,dtype,groups", [(8, "f32", [17]), (10, "bf16", [21]), (20, "f32", [40, 1])])
def test_filter_gradients_of_many_layers(blocks, dtype, groups):
    """One launch holds up to 40 layers; in the fixed order of sums they go through the general kernels, 16 at a time.  From the device's own
    operands (as stored, so that bf16 is as exact as fp32) in float64."""
    import torch
    from oracle import lpref
    from tests.helpers import rel_err
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    say("case many layers", blocks, dtype)
    net = cfg._assemble("deep", [[Block("basic", 16, 16, 16, 1, False)] * blocks], 4, 8, 8, 3, 1, 16, 5, seed=67)
    net.dtype = dtype
    params, _, labels, xs, _ = seeded_step_inputs(net)
    ls = LocalStep(net, keep_gradients=True)
    try:
        ls.set_params(0, params[0])
        ls.set_x(0, xs[0])
        ls.set_labels(labels)
        for fixed in (0, 1):
            B.lp_net_set_deterministic(ls.net, fixed)
            B.lp_profile_enable(ls.net, 2)
            ls.local_step(net.rho, 1.0)
            torch.cuda.synchronize()
            recs = [r["nprob"] for r in B.lp_profile_fetch(ls.net) if r["kind"] == FOLDED_WGRAD]
            B.lp_profile_enable(ls.net, 0)
            assert fixed or recs == groups, recs
            grads, worst = ls.get_grads(0), 0.0
            for u in ls.units(0):
                want = lpref.conv_wgrad(ls.fetch(u.in_, (u.N, u.H, u.W, u.cin)), ls.fetch(u.dy, (u.N, u.Ho, u.Wo, u.cout)), params[0][u.t_w].shape, u.stride, u.pad)
                worst = max(worst, rel_err(grads[u.t_w], want))
            say(f"    fixed order {fixed}: worst {worst:.1e}")
            assert worst <= 1e-4
    finally:
        ls.close()


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


@pytest.mark.parametrize("batch,classes,width", [
    # as many logit gradients as a compute unit's LDS has room for, one more; both filter gradients, the tiled one's array in the same LDS
    (8, 40600, 16), (8, 40704, 16), (8, 40705, 16), (2, 40704, 8), (2, 40705, 8), (2, 50001, 24)])
def test_many_classes(batch, classes, width):
    say("case many classes", batch, classes, width)
    check_units(cfg._assemble("classes", [[Block("bottleneck", width, width, 8, 1, False)]], batch, 2, 2, width, 0, 0, classes, seed=67))


def step_outputs(net, separate):
    """Tensors of one local step through the specialised kernels, or through those they stand in for; and what was launched."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    params, _, labels, xs, lams = seeded_step_inputs(net)
    B.lp_debug_separate_passes(separate)
    try:
        ls = LocalStep(net)
    finally:
        B.lp_debug_separate_passes(False)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        B.lp_profile_enable(ls.net, 2)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        kinds = {(r["kind"], r["cfg"]) for r in B.lp_profile_fetch(ls.net)}
        B.lp_profile_enable(ls.net, 0)
        exact = {f"{n}{k}": t.clone() for n, ts in (("y", ls.y), ("dy", ls.dy), ("dx", ls.dx[1:])) for k, t in enumerate(ts)}
        exact.update(logits=ls.logits.clone(), dlogits=ls.dlogits.clone())
        sums = {}
        for k in range(net.K):
            for i, (info, spec) in enumerate(zip(ls.tables[k], cfg.module_tensor_specs(net.modules[k]))):
                o = info.grad_offset // 4
                g = ls.dparams[k][o:o + int(info.numel)].clone()
                (exact if spec.kind.startswith("bn") else sums)[f"m{k}.{spec.name}"] = g
    finally:
        ls.close()
    return exact, sums, kinds


def assert_same_bits(net, used):
    """Everything but the filter gradients (their partial sums meet in atomics) has the bits of the kernels stood in for."""
    import torch
    got, got_sums, kinds = step_outputs(net, False)
    want, want_sums, general = step_outputs(net, True)
    assert used in kinds and used not in general, (kinds, general)
    differ = {n: int((got[n] != want[n]).sum()) for n in got if not torch.equal(got[n], want[n])}
    say(f"    {len(got)} tensors, differing: {differ}")
    assert all(torch.isfinite(t.float()).all() for t in got.values())
    assert not differ, differ
    for n, g in got_sums.items():                  # fp32 sums of up to 2^17 products in two orders
        assert float((g - want_sums[n]).abs().max()) <= 1e-4 * float(want_sums[n].abs().max()), n


@pytest.mark.parametrize("case", [
    # every width, images of more and of half a tile; 32 samples and more, or modules of more than three blocks
    dict(batch=32, side=(32, 32)), dict(batch=33, side=(32, 32)), dict(batch=3, side=(32, 32), split=[4]),
    dict(batch=128, side=(32, 32), widths=(16, 32)), dict(batch=40, side=(16, 16), widths=(32, 64)), dict(batch=34, side=(8, 8), widths=(64,), stride=1),
    dict(batch=32, side=(32, 32), flags=True),
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", ""))
def test_ordered_tiles_have_the_bits_of_the_separate_passes(case):
    say("case ordered tiles", case)
    assert_same_bits(narrow_net(dtype="bf16", **case), (FOLDED, 0))


@pytest.mark.parametrize("case", [
    # slabs of 64 channels and a half one (160: odd workgroups start there), of 32 (strided layers of 160), 1x1, all tile variants
    dict(batch=1, side=(8, 8), widths=(160, 320)), dict(batch=3, side=(8, 8), widths=(320, 640)), dict(batch=6, side=(16, 16), widths=(160, 320)),
    dict(batch=2, side=(12, 20), widths=(160, 320)), dict(batch=3, side=(14, 14), widths=(640, 1280), kind="bottleneck"),
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", ""))
def test_small_tiles_have_the_bits_of_the_large_ones(case):
    say("case small tiles, bits", case)
    assert_same_bits(wide_net(**case), (CONV, SMALL_TILES))


@pytest.mark.parametrize("lanes", [None, [0, 1], [2, 1], [3, 3]])
def test_narrow_stream_lanes(lanes):
    """The folded passes with the modules on streams of their own."""
    from tests.gpu_common import compare_step
    say("case narrow, stream lanes", lanes)
    compare_step(narrow_net(batch=3, side=(16, 16)), lanes=lanes)


@pytest.mark.parametrize("fixed_forward", [False, True])
def test_fixed_order_switched_between_the_passes(fixed_forward):
    """A forward pass leaves what either backward pass needs: the folded one, or that of the fixed order."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.helpers import rel_err
    say("case fixed order switched, forward", fixed_forward)
    net = narrow_net(batch=3, side=(12, 20))
    params, _, labels, xs, lams = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        for k in range(net.K):
            ls.set_params(k, params[k])
            ls.set_x(k, xs[k])
        ls.set_lams(lams)
        ls.set_labels(labels)
        grads = []
        for switch in (False, True):
            ls.ws.zero_()
            B.lp_net_set_deterministic(ls.net, fixed_forward)
            ls.module_forward()
            ls.local_loss_grad(net.rho, 1.0)
            if switch:
                B.lp_net_set_deterministic(ls.net, not fixed_forward)
            ls.module_backward()
            torch.cuda.synchronize()
            grads.append([g.cpu().numpy() for g in ls.dparams + ls.dx[1:]])
    finally:
        ls.close()
    for a, b in zip(*grads):                       # two orders of the same fp32 sums
        assert rel_err(a, b) <= 1e-4


IMAGE_LAYERS = 31


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,side,stride,c_img", [
    # tiles of whole images and of parts; images that end inside a tile; rows that are no power of two; one and two channels
    (5, (32, 32), 2, 3), (1, (8, 8), 2, 3), (9, (12, 20), 2, 3), (4, (7, 9), 1, 3), (2, (12, 4), 2, 1), (3, (6, 14), 1, 2), (3, (40, 64), 2, 3),
    # an odd number of elements: bf16 images end inside the copy's unit and stay with the general kernel
    (3, (7, 9), 1, 3)])
def test_image_layers_have_the_bits_of_the_general_kernel(batch, side, stride, c_img, dtype):
    """AuxNets of every width in one launch; results in a fixed order go to the general kernel, a launch for each tile."""
    import torch
    import workloads as wl
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    say("case image layers", batch, side, stride, c_img, dtype)
    net = narrow_net(batch, side, dtype=dtype, stride=stride, c_img=c_img, split=[1, 1, 1, 1])
    net.aux = [cfg.AuxDesc(cin=c_img, cout=m.C, stride=net.modules[0].H // m.H, relu=False) for m in net.modules[1:]]
    results = []
    for separate, fixed in ((True, False), (False, False), (False, True)):
        B.lp_debug_separate_passes(separate)
        try:
            ls = LocalStep(net)
        finally:
            B.lp_debug_separate_passes(False)
        try:
            B.lp_net_set_deterministic(ls.net, fixed)
            for j in range(net.K - 1):
                ls.set_aux_params(j, wl.make_aux_params(net, j))
            ls.set_x(0, wl.make_image(net))
            B.lp_profile_enable(ls.net, 2)
            ls.auxnet_forward()
            torch.cuda.synchronize()
            convs = [r["cfg"] for r in B.lp_profile_fetch(ls.net) if r["kind"] == CONV]
            B.lp_profile_enable(ls.net, 0)
            results.append([t.clone() for t in ls.x[1:]])
        finally:
            ls.close()
        whole = batch * side[0] * side[1] * c_img * (4 if dtype == "f32" else 2) % 4 == 0
        assert (convs == [IMAGE_LAYERS]) == (whole and not separate and not fixed), convs
    assert all(float(t.float().abs().max()) > 0 for t in results[0])
    assert all(torch.equal(a, b) for a, b in zip(results[0], results[1]))
    # a fixed order sums the statistics of the stored results in another one: the last place of fp32, a rounding of bf16
    for a, b in zip(results[0], results[2]):
        assert float((a.float() - b.float()).abs().max()) <= (2.0 ** -20 if dtype == "f32" else 2.0 ** -7) * float(a.float().abs().max())


@pytest.mark.parametrize("order,widths,batch,side,c_img,dtype", [
    ("pre", (16, 32), 5, (12, 20), 3, "f32"), ("pre", (16, 64), 3, (32, 32), 3, "bf16"), ("pre", (32, 64), 2, (6, 14), 1, "f32"), ("pre", (64, 16), 2, (8, 8), 2, "bf16"),
    # (images wider than a row of the folded tiles)
    ("post", (16, 32), 2, (4, 72), 3, "f32"), ("post", (64, 16), 3, (2, 80), 3, "bf16"), ("pre", (16, 160), 2, (8, 8), 3, "bf16"),
    ("post", (16, 160), 2, (8, 8), 3, "bf16"), ("post", (64, 128), 3, (12, 4), 3, "f32")])
def test_stems_outside_the_folded_passes(order, widths, batch, side, c_img, dtype):
    """The stem of a network whose batch norms run in passes of their own takes the image-facing kernel too, except in front of wide layers of the
    conv-BN-ReLU order."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    say("case stems", order, widths, batch, side, c_img, dtype)
    net = cfg.with_order(narrow_net(batch, side, widths=widths, dtype=dtype, c_img=c_img, split=[len(widths), 1]), order)
    params, _, _, xs, _ = seeded_step_inputs(net)
    results = []
    for separate in (False, True):
        B.lp_debug_separate_passes(separate)
        try:
            ls = LocalStep(net)
        finally:
            B.lp_debug_separate_passes(False)
        try:
            for k in range(net.K):
                ls.set_params(k, params[k])
                ls.set_x(k, xs[k])
            B.lp_profile_enable(ls.net, 2)
            ls.module_forward()
            torch.cuda.synchronize()
            convs = [r["cfg"] for r in B.lp_profile_fetch(ls.net) if r["kind"] == CONV]
            B.lp_profile_enable(ls.net, 0)
            assert (IMAGE_LAYERS in convs) == (not separate and (order == "pre" or max(b.cout for b in net.modules[0].blocks) <= 64)), convs
            results.append([ls.y[0].clone(), ls.logits.clone()])
        finally:
            ls.close()
    assert float(results[0][0].float().abs().max()) > 0
    for a, b in zip(*results):
        assert torch.equal(a, b)
