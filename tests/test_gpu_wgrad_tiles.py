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

WGRAD, TILE, STEM = 10, 9, 10


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
