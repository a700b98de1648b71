"""First layers whose channels fill no 16-byte vector, against the oracle:
kernel rows of 1 to 33 contiguous elements (under, at and over one vector, an
odd and an even count, so 2- and 4-byte alignments), windows that leave the
image on every side, images narrower than one wave's pixels, a last weight
row and a last pixel at the end of their tensors, and bands."""
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
