"""First layers whose channels fill no 16-byte vector, against the oracle:
kernel rows of 1 to 33 contiguous elements (under, at and over one vector, an
odd and an even count, so 2- and 4-byte alignments), windows that leave the
image on every side, images narrower than one wave's pixels, a last weight
row and a last pixel at the end of their tensors, and bands. And residual
blocks on such maps, where the add is computed in the convolution's epilogue."""
import pytest

from gpu_harness import assert_parity, gpu_run
from paper_2401_11471_amd import lrcnn as L
from workloads import BF16, F32, Inputs, NetBuilder

pytestmark = pytest.mark.gpu

# (channels, kernel, stride, padding, outputs, h, w)
CASES = [
    (3, 7, 2, 3, 24, 37, 61), (3, 7, 2, 3, 70, 20, 150), (3, 3, 1, 1, 8, 19, 23),
    (1, 1, 1, 0, 8, 9, 40), (1, 3, 1, 1, 5, 12, 9), (2, 4, 2, 0, 16, 18, 66),
    (5, 3, 1, 0, 9, 11, 40), (7, 5, 3, 4, 64, 31, 35), (3, 11, 4, 2, 16, 47, 90),
    (6, 2, 1, 0, 4, 8, 5), (3, 1, 2, 0, 72, 15, 33), (3, 16, 8, 8, 8, 40, 48),
]


@pytest.mark.parametrize("dt", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=["c%dk%ds%dp%dn%d_%dx%d" % c for c in CASES])
def test_first_layer_matches_oracle(case, dt):
    c, k, s, p, n, h, w = case
    print(f"first layer {case}", flush=True)
    nb = NetBuilder()
    nb.conv(0, n, k, s, p, affine=1)
    inp = Inputs(nb.nodes, 2, h, w, c, dt, seed=71)
    assert_parity(nb.nodes, inp, gpu_run(nb.nodes, inp, mode=L.CARRY, nb=3, masks=True))


def _sum_of_two(n, k, s):
    # both branches read the image: the later one computes the add
    nb = NetBuilder()
    a = nb.conv(0, n, k, s, k // 2, affine=1, relu=0)
    nb.sum(a, nb.conv(0, n, 1, s, affine=1, relu=0))
    return nb.nodes


def _projection(n):
    # the projection of the image comes first in node order
    nb = NetBuilder()
    p = nb.conv(0, n, 1, affine=1, relu=0)
    u = nb.conv(0, 8, 3, 1, 1)
    nb.sum(p, nb.conv(u, n, 3, 1, 1, relu=1))
    return nb.nodes


def _inner(n):
    # a few-channel map inside the net, an add without ReLU, then a layer
    nb = NetBuilder()
    v = nb.conv(0, 5, 3, 1, 1)
    w = nb.conv(0, n, 3, 1, 1)
    nb.conv(nb.sum(nb.conv(v, n, 3, 1, 1, relu=0), w, relu=0), 16, 3, 1, 1)
    return nb.nodes


BLOCKS = [("sum16", _sum_of_two(16, 3, 1), 33, 15), ("sum24_s2", _sum_of_two(24, 7, 2), 37, 41),
          ("projection", _projection(16), 24, 19), ("inner", _inner(24), 21, 30),
          ("sum72_wide", _sum_of_two(72, 3, 1), 160, 210)]


@pytest.mark.parametrize("dt", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("run", [dict(nb=3), dict(nb=2, bp_refine=2),
                                 dict(mode=L.RECOMPUTE, nb=2), dict(layerwise=True)],
                         ids=["carry3", "refine", "overlap", "layerwise"])
@pytest.mark.parametrize("net", BLOCKS, ids=[b[0] for b in BLOCKS])
def test_few_channel_branches_and_their_sum(net, run, dt):
    name, nodes, h, w = net
    print(f"first layer sum {name} {run}", flush=True)
    inp = Inputs(nodes, 2, h, w, 3, dt, seed=72)
    assert_parity(nodes, inp, gpu_run(nodes, inp, masks=True, **run))
