"""Filter gradients of the wide layers that are not 3x3 with stride 1 (csrc/lp_wgrad_tile.hip) and of image-facing layers
(csrc/lp_wgrad_stem.hip) where rows, columns and pixel chunks do not fill a tile: units against the oracle's float64 primitives,
at the tolerance of tests/gpu_unitwise.py; the launch records say which kernel ran."""
import pytest

from tests.gpu_common import say
from tests.gpu_unitwise import check_units
from tests.test_gpu_narrow import launches
from workloads import configs as cfg
from workloads.configs import Block

pytestmark = pytest.mark.gpu

WGRAD, WGRAD_3X3, TILE, STEM = 10, 8, 9, 10


def net_of(batch, side, widths, stem=1, stem_cout=16, kind="basic"):
    a, b = widths
    w = (lambda c: c // 4) if kind == "bottleneck" else (lambda c: c)
    blocks = [Block(kind, stem_cout, a, w(a), 1, stem_cout != a), Block(kind, a, b, w(b), 2, True)]
    net = cfg._assemble("wgrad", [blocks[:1], blocks[1:]], batch, side[0], side[1], 3, stem, stem_cout, 7, seed=59)
    net.dtype = "bf16"
    return net


@pytest.mark.parametrize("case", [
    dict(batch=2, side=(2, 6), widths=(72, 136)),                                     # fewer pixels than a stage, widths inside a tile
    dict(batch=3, side=(18, 22), widths=(136, 200), stem_cout=16),                    # rows of 22 pixels in steps of 32
    dict(batch=2, side=(10, 34), widths=(160, 296), stem_cout=32),                    # rows of more than a step
    dict(batch=5, side=(32, 48), widths=(128, 256), stem=2, stem_cout=64, kind="bottleneck"),      # 7x7 stem, stride 2; 1x1 layers
    dict(batch=4, side=(64, 64), widths=(256, 512), stem=2, stem_cout=64, kind="bottleneck"),
    dict(batch=9, side=(14, 30), widths=(64, 72), stem_cout=64),                      # tiles of 64 rows
], ids=lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", ""))
def test_units(case):
    say("case filter gradients", case)
    net = net_of(**case)
    check_units(net, note=f" {case}")
    ran = set(launches(net))
    assert (WGRAD, TILE) in ran and (WGRAD, STEM) in ran, ran


def test_odd_image_rows_keep_the_general_kernel():
    """Image rows of an odd number of elements do not start at four bytes."""
    net = net_of(batch=2, side=(6, 10), widths=(72, 136))
    assert (WGRAD, STEM) in launches(net)
    net = cfg._assemble("odd", [[Block("basic", 16, 72, 72, 1, True)]], 2, 6, 9, 3, 1, 16, 7, seed=59)
    net.dtype = "bf16"
    check_units(net)
    assert (WGRAD, STEM) not in launches(net)


@pytest.mark.parametrize("stride,side,cout", [(4, (32, 224), 64), (4, (56, 200), 32), (4, (24, 212), 16), (2, (16, 224), 64), (2, (12, 256), 32)])
def test_strided_image_facing_layers(stride, side, cout):
    """The filter gradient of an AuxNet with stride 2, and with one that is more than its filter, where a step to the next output row
    leaves image rows out and one column class has no tap: images too wide for the narrow kernel, rows of 50 to 128 outputs.
    Oracle's distillation gradient in its storage-rounding mode, at the tolerance of the other tests of it."""
    import torch
    import workloads as wl
    from oracle import lpref
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.helpers import rel_err, store
    say("case strided image-facing layer", stride, side, cout)
    first = [] if stride == 4 else [Block("basic", 16, cout, cout, 2, True)]
    net = cfg._assemble("strided", [first or [Block("basic", cout, cout, cout, 1, False)], [Block("basic", cout, cout, cout, 1, False)]],
                        3, side[0], side[1], 3, 2 if stride == 4 else 1, cout if stride == 4 else 16, 7, seed=79)
    net.dtype = "bf16"
    m = net.modules[1]
    assert (m.H, m.W) == (side[0] // stride, side[1] // stride)
    net.aux = [cfg.AuxDesc(cin=3, cout=cout, stride=stride, relu=False)]
    image, auxp = wl.make_image(net), wl.make_aux_params(net, 0)
    out = lpref.auxnet_forward(net.aux[0], image, auxp, net.bn_eps, wl.round_bf16)
    target = store(net, out + wl.normal(79, "target", out.shape, 0.5))
    ls = LocalStep(net)
    try:
        ls.set_x(0, image)
        ls.set_aux_params(0, auxp)
        ls.auxnet_forward()
        ls.set_x(1, target)
        B.lp_profile_enable(ls.net, 2)
        ls.auxnet_distill_grad(0.5)
        torch.cuda.synchronize()
        ran = {(r["kind"], r["cfg"]) for r in B.lp_profile_fetch(ls.net)}
        loss, grads = lpref.auxnet_distill_grad(net.aux[0], image, auxp, target, net.bn_eps, 0.5, wl.round_bf16)
        errs = [rel_err(g, r) for g, r in zip(ls.get_aux_grads(0), grads)]
    finally:
        ls.close()
    say("    ", ["%.1e" % e for e in errs])
    assert (WGRAD, STEM) in ran, ran
    assert all(e <= 2e-2 for e in errs), errs


def test_update_with_the_rest_of_a_launch_cut_finer():
    """288 output tiles, each summed by one workgroup, but for the 32 of the second round, which are cut in eight: the parameter update
    in the epilogue is then done by whole tiles at once and by the last of eight workgroups that share a tile's ticket.  Oracle's
    update rule on the gradients of the step, at the tolerance of the other tests of it."""
    import numpy as np
    import torch
    from oracle import lpref
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    from tests.gpu_unitwise import seeded_step_inputs
    from tests.helpers import rel_err
    from tests.test_gpu_parity import _read_like_grads, _read_params
    say("case update, rest cut finer")
    net = cfg._assemble("rest", [[Block("basic", 640, 640, 640, 1, False) for _ in range(3)]], 32, 8, 8, 640, 0, 0, 7, seed=73)
    net.dtype = "bf16"
    check_units(net)
    params, _, labels, xs, _ = seeded_step_inputs(net)
    ls = LocalStep(net)
    try:
        ls.set_params(0, params[0])
        ls.set_x(0, xs[0])
        ls.set_labels(labels)
        vel = [torch.zeros_like(d) for d in ls.dparams]
        ls.set_fused_update(True, 1.0, 0.9, 5e-4, velocity=vel)
        B.lp_profile_enable(ls.net, 2)
        for _ in range(2):
            w, v = _read_params(ls, 0), _read_like_grads(ls, vel, 0)
            ls.local_step(net.rho, 1.0)
            torch.cuda.synchronize()
            got_w, got_v = _read_params(ls, 0), _read_like_grads(ls, vel, 0)
            for i, (info, g) in enumerate(zip(ls.tables[0], ls.get_grads(0))):
                want_w, want_v = lpref.sgd_update(w[i], g.astype(np.float64), 1.0, v[i], 0.9, 5e-4)
                tol = 4e-3 if info.dtype == B.LP_BF16 else 1e-6              # one rounding of the stored value
                assert rel_err(got_w[i], want_w) <= tol and rel_err(got_v[i], want_v) <= 1e-6, i
                assert np.max(np.abs(want_w - w[i])) >= 5 * tol * np.max(np.abs(want_w)), i       # a missing update would show
        blocks = [(r["nprob"], r["blocks"]) for r in B.lp_profile_fetch(ls.net) if (r["kind"], r["cfg"]) == (WGRAD, WGRAD_3X3)]
    finally:
        ls.close()
    assert blocks == [(6, 256 + 32 * 8)] * 2, blocks
