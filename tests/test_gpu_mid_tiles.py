"""The implicit-GEMM tiles with waves of 32 pixels (csrc/lp_conv_fast.hip): rows and channels that do not fill the last tile,
strides, 1x1 layers, added skip gradients, every ring depth.  Units against the oracle's float64 primitives, at the tolerance of
tests/gpu_unitwise.py; the launch records say which tiles ran."""
import pytest

from tests.gpu_common import say
from tests.gpu_unitwise import check_units
from tests.test_gpu_narrow import CONV, SMALL_TILES, assert_same_bits, launches
from workloads import configs as cfg
from workloads.configs import Block

pytestmark = pytest.mark.gpu

T128, T128_R3, T128x32, T64, T64x64, T128x64, T128x64_R3, T256, T256x64, T256x32 = 17, 18, 19, 20, 25, 26, 27, 28, 29, 30


def net_of(batch, side, widths, kind="basic"):
    a, b = widths
    w = (lambda c: c // 4) if kind == "bottleneck" else (lambda c: c)
    blocks = [Block(kind, a, a, w(a), 1, False), Block(kind, a, b, w(b), 2, True), Block(kind, b, b, w(b), 1, False)]
    net = cfg._assemble("mid", [blocks[:1], blocks[1:]], batch, side[0], side[1], 3, 1, a, 7, seed=53)
    net.dtype = "bf16"
    return net


CASES = [
    (dict(batch=1, side=(4, 6), widths=(64, 128)), {T64x64, T256x32}),                # fewer rows than a tile
    (dict(batch=5, side=(14, 10), widths=(192, 320)), {T128x32}),                     # widths that end inside a tile, rows too
    (dict(batch=3, side=(28, 28), widths=(256, 512), kind="bottleneck"), {T64, T64x64, T128x64_R3, T256x64, T256x32}),
    (dict(batch=20, side=(28, 28), widths=(256, 512), kind="bottleneck"), {T128, T128_R3, T64, T64x64, T256, T256x64}),
    (dict(batch=40, side=(30, 26), widths=(64, 192)), {T128x64_R3}),
    (dict(batch=24, side=(16, 16), widths=(320, 640)), {T128_R3, T128x64_R3, T256x64}),
    (dict(batch=40, side=(40, 40), widths=(256, 256), kind="bottleneck"), {T128, T128x64}),
]
ids = lambda c: "-".join(f"{k}{v}" for k, v in c.items()).replace(" ", "") if isinstance(c, dict) else ""      # noqa: E731


@pytest.mark.parametrize("case,tiles", CASES, ids=ids)
def test_units(case, tiles):
    say("case mid tiles", case)
    net = net_of(**case)
    check_units(net, note=f" {case}")
    ran = {c for k, c in launches(net) if k == CONV}
    assert tiles <= ran, ran


@pytest.mark.parametrize("case,tiles", CASES, ids=ids)
def test_bits_of_the_large_tiles(case, tiles):
    """Every output of a step, batch statistics included, is the one of the tiles these stand in for, bit for bit."""
    say("case mid tiles, bits", case)
    assert_same_bits(net_of(**case), (CONV, min(tiles)))


@pytest.mark.parametrize("batch,side,width", [(8, 8, 320), (1, 14, 256), (1, 16, 320), (1, 28, 256), (6, 14, 256), (1, 8, 160), (3, 8, 640), (2, 32, 192)])
def test_query_names_the_kernel_that_runs(batch, side, width):
    """The host's answer for a layer alone in its launch against the launch records of a network of one block (both forward
    layers, with their batch statistics, and the second one's data gradient)."""
    import torch
    from paper_2112_05387_amd import LocalStep
    from paper_2112_05387_amd import binding as B
    say("case layer query", batch, side, width)
    net = cfg._assemble("query", [[Block("basic", width, width, width, 1, False)]], batch, side, side, width, 0, 0, 7, seed=71)
    net.dtype = "bf16"
    want = B.lp_debug_layer_kernels("bf16", batch, side, side, width, width, 3, 1)
    ls = LocalStep(net)
    try:
        B.lp_profile_enable(ls.net, 2)
        ls.local_step(net.rho, 1.0)
        torch.cuda.synchronize()
        small = [r["cfg"] == SMALL_TILES for r in B.lp_profile_fetch(ls.net) if r["kind"] == CONV]
    finally:
        ls.close()
    assert small == [want["small_fwd"], want["small_fwd"], want["small_dgrad"]], (small, want)
