"""Batch-norm apply passes whose workgroups have a slice of the channels (csrc/lp_kernels.h: bn_slice): slices of 64 and 128
channels, one and several of them, rows that do not fill a workgroup, projections and added gradients, and tensors either side of
the size from which a thread takes two trips of loads.  Units against the oracle's float64 primitives."""
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
