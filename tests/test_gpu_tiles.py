"""Convolution tiles at their edges, against the oracle: maps of one pixel
less than, exactly and one more than a 64- or 128-pixel tile (and a single
pixel), output and input channels around 64, K of one and of several steps,
so that small, narrow and wide tiles end on and off their last row, column
and step, forward and input gradient; and maps large enough that the band,
layer-wise and tail launches of one layer take different tiles (their
outputs must be equal bit for bit: gpu_run compares them)."""
import pytest

from gpu_harness import assert_parity, gpu_run
from paper_2401_11471_amd import lrcnn as L
from workloads import BF16, F32, Inputs, NetBuilder

pytestmark = pytest.mark.gpu

# (h, w, channels in, kernel, channels out)
CASES = [
    (1, 1, 64, 1, 64), (7, 9, 64, 1, 72), (8, 8, 8, 3, 64), (5, 13, 72, 3, 56),
    (1, 127, 256, 1, 8), (8, 16, 64, 3, 128), (3, 43, 136, 1, 200), (26, 5, 16, 3, 264),
    (96, 130, 64, 1, 64), (64, 200, 64, 3, 72),
]


@pytest.mark.parametrize("dt", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=["%dx%d_c%dk%dn%d" % c for c in CASES])
def test_tile_edges_match_oracle(case, dt):
    h, w, ci, k, n = case
    print(f"tiles {case}", flush=True)
    nb = NetBuilder()
    u = nb.conv(0, n, k, 1, k // 2, affine=1)
    nb.conv(u, ci, k, 1, k // 2, relu=0)
    inp = Inputs(nb.nodes, 1 if h < 50 else 2, h, w, ci, dt, seed=81)
    for kw in (dict(nb=1), dict(nb=min(h, 3)), dict(layerwise=True)):
        assert_parity(nb.nodes, inp, gpu_run(nb.nodes, inp, want_dx=True, masks=True, **kw))


@pytest.mark.parametrize("dt", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("c,kh,s,p", [(8, 2, 2, 0), (12, 3, 2, 1), (5, 3, 1, 1), (64, 5, 3, 2)])
def test_pool_vectors_match_oracle(c, kh, s, p, dt):
    # 16-byte, 8-byte and single-element channel vectors
    nb = NetBuilder()
    u = nb.conv(0, c, 1, affine=1, relu=0)
    nb.pool(u, kh, s, p)
    inp = Inputs(nb.nodes, 2, 21, 17, 3, dt, seed=83)
    for kw in (dict(nb=4), dict(mode=L.RECOMPUTE, nb=3)):
        assert_parity(nb.nodes, inp, gpu_run(nb.nodes, inp, want_dx=True, masks=True, **kw))
