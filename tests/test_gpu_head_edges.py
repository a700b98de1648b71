"""Classifier head and update at the edges of their splits, against float64:
features that fill one, two or four-wide accesses and end on, before or
after a 2048-feature chunk, the fewest and most classes, more images and
classes than one block has threads, and an update of more tensors than one
launch takes, with weights shared by two layers (updated twice, in order). And
gradients written over the inputs they do not need any more."""
import numpy as np
import pytest
import torch

from oracle import head as OH
from paper_2401_11471_amd import lrcnn as L
from workloads import BF16, F32, NetBuilder

pytestmark = pytest.mark.gpu


def _plan(batch, k, dtype):
    nb = NetBuilder()
    nb.conv(0, k, 1)
    return L.lrcnn_plan(nb.nodes, batch, 8, 1, 1, dtype)


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("batch,k,classes", [
    (1, 5, 1), (3, 12, 64), (5, 2048, 10), (2, 2049, 3), (2, 2052, 64), (33, 4100, 17),
    (300, 260, 2), (8, 25088, 10)])
def test_head_edges(batch, k, classes, dtype):
    print(f"head {batch} {k} {classes}", flush=True)
    plan = _plan(batch, k, dtype)
    rng = np.random.default_rng(k)
    tdt = torch.bfloat16 if dtype == BF16 else torch.float32
    y = torch.from_numpy(rng.standard_normal((batch, 1, 1, k), dtype=np.float32)).cuda().to(tdt)
    fw = (rng.standard_normal((classes, k)) / np.sqrt(k)).astype(np.float32)
    fb = rng.standard_normal(classes).astype(np.float32)
    lab = rng.integers(0, classes, batch).astype(np.int32)

    def dev(a):
        return torch.from_numpy(a).cuda()

    def out(*s):
        return torch.full(s, float("nan"), device="cuda")
    logits, loss, dfw, dfb = out(batch, classes), out(4), out(classes, k), out(classes)
    dy = torch.full_like(y, float("nan"))
    ws = torch.empty(L.lrcnn_head_workspace_bytes(plan, classes), dtype=torch.uint8, device="cuda")
    L.lrcnn_head_loss(plan, y, dev(fw), dev(fb), dev(lab), logits, loss, dy, dfw, dfb, ws)
    torch.cuda.synchronize()
    yn = y.float().cpu().numpy()
    rl = OH.head_forward(yn, fw, fb)
    rloss, dlog = OH.softmax_xent(rl, lab)
    rdy, rdfw, rdfb = OH.head_backward(yn, fw, dlog)

    def rel(a, r):
        return float(np.abs(a.float().cpu().numpy() - r).max() / max(np.abs(r).max(), 1e-30))
    # sums of up to 25088 float32 products in tree order: a few 1e-7; the
    # largest bfloat16 rounding is 2^-8
    assert rel(logits, rl) < 1e-5
    assert abs(loss[0].item() - rloss) <= 1e-5 * max(abs(rloss), 1e-2)
    if classes > 1:
        assert rel(dfw, rdfw) < 1e-5 and rel(dfb, rdfb) < 1e-5
        assert rel(dy, rdy) < (1e-5 if dtype == F32 else 2.0 ** -8)


@pytest.mark.parametrize("over", ["dy_over_y", "d_fc_w_over_fc_w"])
@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("batch,k,classes", [(3, 12, 64), (4, 2049, 7), (5, 20000, 10)])
def test_head_gradients_over_inputs(batch, k, classes, dtype, over):
    print(f"head {over} {batch} {k} {classes}", flush=True)
    plan = _plan(batch, k, dtype)
    rng = np.random.default_rng(k + 1)
    tdt = torch.bfloat16 if dtype == BF16 else torch.float32
    y = torch.from_numpy(rng.standard_normal((batch, 1, 1, k), dtype=np.float32)).cuda().to(tdt)
    fw = (rng.standard_normal((classes, k)) / np.sqrt(k)).astype(np.float32)
    fb = rng.standard_normal(classes).astype(np.float32)
    lab = rng.integers(0, classes, batch).astype(np.int32)
    yn = y.float().cpu().numpy()

    def dev(a):
        return torch.from_numpy(a).cuda()
    fcw = dev(fw)
    logits, loss = torch.empty((batch, classes), device="cuda"), torch.empty(4, device="cuda")
    dfb = torch.empty(classes, device="cuda")
    dy = y if over == "dy_over_y" else torch.empty_like(y)
    dfw = fcw if over == "d_fc_w_over_fc_w" else torch.empty_like(fcw)
    ws = torch.empty(L.lrcnn_head_workspace_bytes(plan, classes), dtype=torch.uint8, device="cuda")
    L.lrcnn_head_loss(plan, y, fcw, dev(fb), dev(lab), logits, loss, dy, dfw, dfb, ws)
    torch.cuda.synchronize()
    rl = OH.head_forward(yn, fw, fb)
    rloss, dlog = OH.softmax_xent(rl, lab)
    rdy, rdfw, rdfb = OH.head_backward(yn, fw, dlog)

    def rel(a, r):
        return float(np.abs(a.float().cpu().numpy() - r).max() / np.abs(r).max())
    # (the bounds of test_head_edges; with dy over y, d_fc_w has no y left)
    assert rel(logits, rl) < 1e-5
    assert abs(loss[0].item() - rloss) <= 1e-5 * max(abs(rloss), 1e-2)
    assert rel(dfb, rdfb) < 1e-5
    assert rel(dy, rdy) < (1e-5 if dtype == F32 else 2.0 ** -8)
    if over != "dy_over_y":
        assert rel(dfw, rdfw) < 1e-5


@pytest.mark.parametrize("dtype", [F32, BF16], ids=["f32", "bf16"])
def test_update_of_many_and_shared_tensors(dtype):
    nb = NetBuilder()
    v = 0
    for i in range(30):
        v = nb.conv(v, 7 if i % 2 else 9, 3, 1, 1)
    plan = L.lrcnn_plan(nb.nodes, 1, 9, 4, 4, dtype)
    tdt = torch.bfloat16 if dtype == BF16 else torch.float32
    gen = torch.Generator("cuda").manual_seed(3)
    ch = [9] + [nd[3] for nd in nb.nodes[1:]]
    w, g = [None], [None]
    for i in range(30):
        shape = (ch[i + 1], 3, 3, ch[i])
        w.append(torch.randn(shape, generator=gen, device="cuda").to(tdt))
        g.append(torch.randn(shape, generator=gen, device="cuda"))
    w[6] = w[4]  # shared by two layers
    lr = 0.25
    want = [None if t is None else t.clone() for t in w]
    want[6] = want[4]
    for i in range(1, 31):
        want[i].copy_((want[i].double() - lr * g[i].double()).float().to(tdt))
    L.lrcnn_sgd_update(plan, lr, w, g)
    torch.cuda.synchronize()
    for i in range(1, 31):
        # one float32 rounding (one storage rounding) per update
        err = (w[i].double() - want[i].double()).abs().max().item()
        assert err <= 8 * (2.0 ** -23 if dtype == F32 else 2.0 ** -8), i
