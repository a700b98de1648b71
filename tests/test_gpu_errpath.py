"""Where the errors of a block's branches leave and enter a band, on blocks
alone (so the block's add or pooling is also the output node, whose error is
dL/dy read in place), against the oracle: a projection branch that owns its
rows a band earlier than the add reads them (its carried errors leave with
the add's backward; the other branch computes the add), windows whose last
row no consumer row of the band reaches (odd rows before a stride-2
pooling or convolution), and inputs whose error nobody wants."""
import pytest

from gpu_harness import assert_parity, gpu_run
from paper_2401_11471_amd import lrcnn as L
from workloads import BF16, F32, Inputs, NetBuilder

pytestmark = pytest.mark.gpu


def _block(stride, project, c):
    nb = NetBuilder()
    u = nb.conv(0, 8, 1, affine=1)
    u = nb.conv(u, 8, 3, stride, 1, affine=1)
    u = nb.conv(u, c, 1, affine=1, relu=0)
    v = nb.conv(0, c, 1, stride, affine=1, relu=0) if project else 0
    nb.sum(u, v)
    return nb.nodes


def _stem(c):
    nb = NetBuilder()
    v = nb.conv(0, c, 7, 2, 3, affine=1)
    nb.pool(v, 3, 2, 1)
    return nb.nodes


# (name, nodes, input channels): 24 channels fill 16-byte vectors, 12 only
# 8-byte ones in bfloat16, 6 none at all
NETS = [
    ("project", _block(1, True, 24), 16),
    ("project_s2", _block(2, True, 24), 16),
    ("identity", _block(1, False, 24), 24),
    ("identity_c12", _block(1, False, 12), 12),
    ("project_c6", _block(1, True, 6), 8),
    ("stem", _stem(24), 3),
    ("stem_c6", _stem(6), 3),
]
RUNS = [
    ("carry5", dict(mode=L.CARRY, nb=5)),
    ("carry_odd", dict(mode=L.CARRY, nb=4, policy=L.EXPLICIT, bounds=[0, 7, 12, 13, 33])),
    ("refine", dict(mode=L.CARRY, nb=2, bp_refine=3)),
    ("overlap", dict(mode=L.RECOMPUTE, nb=3)),
    ("layerwise", dict(layerwise=True)),
]


@pytest.mark.parametrize("dt", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("run", RUNS, ids=[r[0] for r in RUNS])
@pytest.mark.parametrize("net", NETS, ids=[n[0] for n in NETS])
def test_block_errors_match_oracle(net, run, dt):
    name, nodes, c = net
    print(f"block errors {name} {run[0]}", flush=True)
    inp = Inputs(nodes, 2, 33, 15, c, dt, seed=61)
    for dx in (True, False):
        assert_parity(nodes, inp, gpu_run(nodes, inp, want_dx=dx, masks=True, **run[1]),
                      check_dx=dx)
