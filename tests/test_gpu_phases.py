"""Input gradient of strided convolutions split into stride phases (producer
rows and columns grouped by (y + pad) mod s, each phase dense with only the
taps that reach it), all in one launch, in launches of their own, and by
estimate, against the single launch over all taps, and against the float64
oracle. Odd map sizes give phases of unequal
size; a 1x1 stride-2 convolution has phases without taps."""
import numpy as np
import pytest

from gpu_harness import assert_parity, gpu_run, rel
from paper_2401_11471_amd import lrcnn as L
from workloads import BF16, F32, Inputs, NetBuilder, resnet50_net

pytestmark = pytest.mark.gpu


def strided_net(last_pad=0):
    nb = NetBuilder()
    v = nb.conv(0, 16, 7, 2, 3, affine=1)       # stem-like, 3 input channels
    v = nb.conv(v, 32, 3, 2, 1)                  # 3x3 stride 2, pad 1
    a = nb.conv(v, 32, 1, 2, 0, relu=0)          # 1x1 stride 2 (phases without taps)
    b = nb.conv(v, 32, 3, 2, 1, relu=0)
    v = nb.sum(a, b)
    # stride 2 without padding leaves rows no output reads, which
    # overlapping partitioning never computes (their masks stay unwritten)
    v = nb.conv(v, 48, 3, 2, last_pad)
    return nb.nodes


def strided_net_padded():
    return strided_net(1)


def _run(nodes, inp, phases, **kw):
    L.lrcnn_debug_dgrad_phases(phases)
    try:
        return gpu_run(nodes, inp, **kw)
    finally:
        L.lrcnn_debug_dgrad_phases(0)


CASES = [
    ("strided_f32_carry3", strided_net, F32, 2, 75, 61, dict(mode=L.CARRY, nb=3)),
    ("strided_bf16_recompute2", strided_net_padded, BF16, 2, 75, 61,
     dict(mode=L.RECOMPUTE, nb=2)),
    ("strided_f32_layerwise", strided_net, F32, 1, 69, 53, dict(layerwise=True)),
    ("resnet50_f32_carry2", resnet50_net, F32, 1, 96, 64, dict(mode=L.CARRY, nb=2)),
    ("resnet50_bf16_carry3", resnet50_net, BF16, 2, 96, 96, dict(mode=L.CARRY, nb=3)),
]


@pytest.mark.parametrize("name,net,dt,b,h,w,kw", CASES, ids=[c[0] for c in CASES])
def test_phased_input_gradient(name, net, dt, b, h, w, kw):
    print(f"dgrad phases {name}", flush=True)
    nodes = net()
    inp = Inputs(nodes, b, h, w, 3, dt, seed=21)
    one = _run(nodes, inp, 2, want_dx=True, **kw)
    for mode in (1, 3, 4):
        ph = _run(nodes, inp, mode, want_dx=True, **kw)
        # the forward is untouched; the backward agrees with the single launch
        # to rounding (split-K groupings may differ)
        assert np.array_equal(ph["y"], one["y"])
        tol = 2e-2 if dt == BF16 else 1e-5
        assert rel(ph["dx"], one["dx"]) < tol, mode
        for v, (p, q) in enumerate(zip(ph["dw"], one["dw"])):
            if p is not None:
                assert rel(p, q) < tol, (mode, v)
        assert_parity(nodes, inp, ph)
