"""Performance cases of the row-centric training library.

Each case is one call sequence of a user's program through the public entry
points: a plan and its buffers are made once (``prepare``), then a pass
(``run``) is a forward, a training step (forward and backward), a layer-wise
step, an allocation-free forward, or a full step with classifier head and
SGD. ``exact`` computes the same outputs in float64 with plain torch.

The whole networks are those of the repository's workloads (the tiny 3x3
stack, VGG-16, ResNet-50). Most cases are single blocks of them, at the map
sizes and band counts the block has inside the two high-resolution and the
two 224-pixel workloads, because a block can be compared far more tightly
than a whole bfloat16 network: a rounding that differs in one layer decides
ReLUs differently in all the layers after it.
"""
from __future__ import annotations

import math

import torch

from paper_2401_11471_amd import lrcnn as L
from paper_2401_11471_amd.device import DeviceModel
from paper_2401_11471_amd.train import Trainer
from workloads import NetBuilder, resnet50_net, tiny_net, vgg16_net

CONV, POOL = L.OP_CONV, L.OP_MAXPOOL
LR = 1e-5
CLASSES = 10

# Every key of a case:
#   net     tiny | vgg16 | resnet50 | chain | bottleneck | stem | head
#   call    step (forward_rows + backward_rows) | forward (forward_rows) |
#           static (forward_rows_static) | layerwise | train (Trainer.step)
#   bf16    storage type of the maps (else float32)
#   batch, h, w, c   the input
#   width, convs, pool, stride, project   the block (where the net has them)
#   bands, refine, balanced, recompute, hybrid   the plan
#   dx      dL/dx is wanted too
_DEFAULTS = dict(bf16=False, width=0, convs=0, pool=False, stride=1, project=False,
                 bands=1, refine=1, balanced=False, recompute=False, hybrid=False, dx=False)


def _case(**kw):
    return dict(_DEFAULTS, **kw)


def listed():
    return [
        # the smallest step: three 3x3 convolutions of 8 channels on one
        # 32 x 32 image in 4 bands; launches and their latency decide
        _case(name="tiny_f32_step", net="tiny", call="step", batch=1, h=32, w=32, c=3,
              width=8, convs=3, bands=4, dx=True),
        # serving without allocation: ResNet's stem and first block on one
        # 224-pixel image, through the library's own workspace
        _case(name="stem_block_bf16_static", net="head", call="static", bf16=True, batch=1,
              h=224, w=224, c=3, width=64, bands=2),
        # the 224-pixel VGG-16 workload with its preset: a whole float32
        # training step (4 forward bands, 8 backward bands, a checkpoint)
        _case(name="vgg16_f32_224_step", net="vgg16", call="step", batch=8, h=224, w=224, c=3,
              bands=4, refine=2, hybrid=True),
        # the 224-pixel ResNet-50 workload: a whole forward with the
        # planner's checkpoint (evaluation between training steps)
        _case(name="resnet50_bf16_224_fwd", net="resnet50", call="forward", bf16=True, batch=16,
              h=224, w=224, c=3, bands=8, hybrid=True),
        # ResNet-50 on 2400 x 3600 images in 32 bands, block by block: the
        # 7x7 stride-2 stem with its pooling
        _case(name="stem_bf16_2400x3600", net="stem", call="step", bf16=True, batch=8, h=2400,
              w=3600, c=3, width=64, bands=32),
        # its first block, with projection, on 600 x 900 maps: memory-bound
        # 1x1 convolutions
        _case(name="block1_bf16_600x900", net="bottleneck", call="step", bf16=True, batch=8,
              h=600, w=900, c=64, width=64, project=True, bands=32),
        # the first block of its third stage: stride 2, an odd width after it
        _case(name="block3_bf16_300x450_s2", net="bottleneck", call="step", bf16=True, batch=8,
              h=300, w=450, c=512, width=256, stride=2, project=True, bands=32),
        # a block of its last stage on 75 x 113 maps: two or three rows a
        # band, many small launches
        _case(name="block4_bf16_75x113", net="bottleneck", call="step", bf16=True, batch=8,
              h=75, w=113, c=2048, width=512, bands=32),
        # VGG-16 in float32 on 1200 x 1800 images in 16 bands: its third
        # block, three 3x3 convolutions and the pooling, with dL/dx
        _case(name="conv3_f32_300x450", net="chain", call="step", batch=4, h=300, w=450, c=128,
              width=256, convs=3, pool=True, bands=16, dx=True),
        # overlapping partitioning (RECOMPUTE) of two bfloat16 3x3 layers,
        # with dL/dx
        _case(name="conv4_bf16_56x56_overlap", net="chain", call="step", bf16=True, batch=8,
              h=56, w=56, c=256, width=512, convs=2, bands=4, recompute=True, dx=True),
        # the layer-wise step (no row partition) of a second-stage block at
        # 224-pixel size
        _case(name="block2_bf16_28x28_layerwise", net="bottleneck", call="layerwise", bf16=True,
              batch=16, h=28, w=28, c=512, width=128),
        # a full float32 training step on VGG-16's last block: row-centric
        # forward and backward, classifier head, loss and SGD update
        _case(name="conv5_f32_14x14_train", net="chain", call="train", batch=8, h=14, w=14,
              c=512, width=512, convs=3, pool=True, bands=2),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fit(case, pixels):
    """Shrinks a drawn map so that batch x h x w stays below `pixels`."""
    while case["batch"] * case["h"] * case["w"] > pixels:
        if case["batch"] > 1:
            case["batch"] -= 1
        else:
            case["h"], case["w"] = max(8, case["h"] * 3 // 4), max(8, case["w"] * 3 // 4)
    case["bands"] = max(1, min(case["bands"], case["h"] // 2))
    return case


def draw(rng):
    kind = rng.choice(("tiny", "static", "vgg16", "resnet50", "stem", "block", "block",
                       "chain", "chain", "layerwise", "train"))
    if kind == "tiny":
        return _case(net="tiny", call="step", bf16=rng.random() < 0.3, batch=rng.randint(1, 4),
                     h=rng.randint(16, 80), w=rng.randint(16, 80), c=3,
                     width=8 * rng.randint(1, 4), convs=rng.randint(2, 4),
                     bands=rng.randint(1, 5), dx=rng.random() < 0.7)
    if kind == "static":
        return _case(net="head", call="static", bf16=rng.random() < 0.7, batch=1,
                     h=rng.randint(64, 256), w=rng.randint(64, 256), c=3, width=64,
                     bands=rng.randint(2, 4))
    if kind == "vgg16":
        return _case(net="vgg16", call="step", batch=rng.randint(1, 8), h=rng.randint(64, 224),
                     w=rng.randint(64, 224), c=3, bands=rng.randint(2, 5),
                     refine=rng.randint(1, 2), hybrid=rng.random() < 0.5)
    if kind == "resnet50":
        return _case(net="resnet50", call="forward", bf16=True, batch=rng.randint(1, 16),
                     h=rng.randint(96, 320), w=rng.randint(96, 320), c=3,
                     bands=rng.randint(2, 8), hybrid=rng.random() < 0.5)
    if kind == "stem":
        return _fit(_case(net="stem", call="step", bf16=rng.random() < 0.8,
                          batch=rng.randint(1, 8), h=_log(rng, 160, 2400),
                          w=_log(rng, 160, 3600), c=3, width=64, bands=_log(rng, 2, 32)),
                    30_000_000)
    if kind in ("block", "layerwise"):
        width = rng.choice((64, 128, 256, 512))
        # maps as large as the stage has them at 2400 x 3600
        big = 600 * 64 // width
        stride = 2 if width > 64 and rng.random() < 0.4 else 1
        project = stride == 2 or rng.random() < 0.3
        c = (64 if width == 64 else 2 * width) if project else 4 * width
        scale = 2 if stride == 2 else 1
        case = _case(net="bottleneck", call="step" if kind == "block" else "layerwise", bf16=True,
                     batch=rng.randint(1, 8), h=_log(rng, 14, scale * big),
                     w=_log(rng, 14, scale * big * 3 // 2), c=c, width=width, stride=stride,
                     project=project)
        if kind == "block":
            case["bands"] = _log(rng, 2, 32)
            case["recompute"] = rng.random() < 0.2
            case["balanced"] = not case["recompute"] and rng.random() < 0.1
        return _fit(case, (4_000_000 if kind == "block" else 1_000_000) * 64 // width)
    if kind == "chain":
        width = rng.choice((64, 128, 256, 512))
        bf16 = rng.random() < 0.4
        big = 1200 * 64 // width
        case = _case(net="chain", call="step", bf16=bf16, batch=rng.randint(1, 8),
                     h=_log(rng, 14, big), w=_log(rng, 14, big * 3 // 2),
                     c=rng.choice((width, max(64, width // 2))), width=width,
                     convs=rng.randint(2, 2 if bf16 else 3), pool=rng.random() < 0.6,
                     bands=_log(rng, 2, 16), recompute=rng.random() < 0.25,
                     refine=rng.randint(1, 2), dx=rng.random() < 0.5)
        return _fit(case, 540_000 * 256 * 256 // (width * width))
    return _case(net="chain", call="train", bf16=False, batch=rng.randint(1, 8),
                 h=rng.randint(8, 56), w=rng.randint(8, 56), c=rng.choice((64, 128, 256, 512)),
                 width=rng.choice((128, 256, 512)), convs=rng.randint(1, 3), pool=True,
                 bands=rng.randint(1, 4))


def _nodes(case):
    net, wd = case["net"], case["width"]
    if net == "tiny":
        return tiny_net((wd,) * case["convs"])
    if net == "vgg16":
        return vgg16_net()
    if net == "resnet50":
        return resnet50_net()
    nb = NetBuilder()
    v = 0
    if net == "chain":
        for _ in range(case["convs"]):
            v = nb.conv(v, wd, 3, 1, 1)
        if case["pool"]:
            v = nb.pool(v, 2, 2)
        return nb.nodes
    if net in ("stem", "head"):
        v = nb.conv(v, wd, 7, 2, 3, affine=1)
        v = nb.pool(v, 3, 2, 1)
        if net == "stem":
            return nb.nodes
    s = case["stride"]
    u = nb.conv(v, wd, 1, affine=1)
    u = nb.conv(u, wd, 3, s, 1, affine=1)
    u = nb.conv(u, 4 * wd, 1, affine=1, relu=0)
    if net == "head" or case["project"]:
        v = nb.conv(v, 4 * wd, 1, s, affine=1, relu=0)
    nb.sum(u, v)
    return nb.nodes


def _channels(nodes, c):
    ch = [c]
    for nd in nodes[1:]:
        ch.append(nd[3] if nd[0] == CONV else ch[nd[1]])
    return ch


def _sizes(nodes, h, w):
    out = [(h, w)]
    for (op, in0, _in1, _c, kh, kw, sh, sw, ph, pw, _a, _r) in nodes[1:]:
        a, b = out[in0]
        out.append(((a + 2 * ph - kh) // sh + 1, (b + 2 * pw - kw) // sw + 1)
                   if op in (CONV, POOL) else (a, b))
    return out


def _inputs(case, seed):
    """x, weights, affine scales and shifts, dL/dy: an image is N(0, 1), a
    block's input is the ReLU of it, weights are He-normal."""
    nodes = _nodes(case)
    gen = torch.Generator("cuda").manual_seed(seed)
    dt = torch.bfloat16 if case["bf16"] else torch.float32
    ch, size = _channels(nodes, case["c"]), _sizes(nodes, case["h"], case["w"])

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    x = normal(case["batch"], case["h"], case["w"], case["c"])
    if case["c"] > 3:
        x.clamp_(min=0)
    ws, scs, sfs = [None], [None], [None]
    for nd in nodes[1:]:
        w = sc = sf = None
        if nd[0] == CONV:
            ci = ch[nd[1]]
            w = (normal(nd[3], nd[4], nd[5], ci) * math.sqrt(2.0 / (ci * nd[4] * nd[5]))).to(dt)
            if nd[10]:
                sc = torch.rand(nd[3], generator=gen, device="cuda") * 0.5 + 0.5
                sf = torch.rand(nd[3], generator=gen, device="cuda") * 0.2 - 0.1
        ws.append(w)
        scs.append(sc)
        sfs.append(sf)
    dy = normal(case["batch"], *size[-1], ch[-1]).to(dt)
    return nodes, x.to(dt), ws, scs, sfs, dy


def _head_inputs(nodes, case, seed):
    """Classifier weights, bias and labels of a full training step."""
    ch, size = _channels(nodes, case["c"]), _sizes(nodes, case["h"], case["w"])
    k = size[-1][0] * size[-1][1] * ch[-1]
    gen = torch.Generator("cuda").manual_seed(seed + 1_000_003)
    fc_w = torch.randn((CLASSES, k), generator=gen, device="cuda") / math.sqrt(k)
    fc_b = torch.zeros(CLASSES, device="cuda")
    labels = torch.randint(0, CLASSES, (case["batch"],), generator=gen, device="cuda")
    return fc_w, fc_b, labels.to(torch.int32)


def prepare(case, seed):
    nodes, x, ws, scs, sfs, dy = _inputs(case, seed)
    plan = L.lrcnn_plan(
        nodes, case["batch"], case["c"], case["h"], case["w"],
        dtype=L.BF16 if case["bf16"] else L.F32,
        mode=L.RECOMPUTE if case["recompute"] else L.CARRY, n_bands=case["bands"],
        policy=L.BALANCED if case["balanced"] else L.EVEN, bp_refine=case["refine"],
        hybrid_from=L.HYBRID_AUTO if case["hybrid"] else 0)
    st = dict(call=case["call"], plan=plan)
    if case["call"] == "train":
        def host(ts):
            return [None if t is None else t.cpu().numpy() for t in ts[1:]]
        dm = DeviceModel(nodes, x.cpu().numpy(), host(ws), host(scs), host(sfs), L.F32)
        st["trainer"] = Trainer(plan, dm, *_head_inputs(nodes, case, seed))
        return st
    info = plan.info()
    need = info["layerwise_workspace_bytes" if case["call"] == "layerwise" else "workspace_bytes"]
    st.update(x=x, w=ws, sc=scs, sf=sfs, y=torch.empty_like(dy))
    if case["call"] != "static":
        st["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    if case["call"] in ("step", "layerwise"):
        st["dy"] = dy
        st["dw"] = [None if w is None else torch.empty(w.shape, device="cuda") for w in ws]
        st["dx"] = torch.empty_like(x) if case["dx"] else None
    return st


def run(st):
    call = st["call"]
    if call == "train":
        tr = st["trainer"]
        loss = tr.step(LR)
        return dict(loss=loss, logits=tr.logits, w=[w for w in tr.dm.w if w is not None],
                    dw=[d for d in tr.dm.dw if d is not None], fc_w=tr.fc_w, fc_b=tr.fc_b,
                    d_fc_w=tr.d_fc_w, d_fc_b=tr.d_fc_b)
    a = (st["plan"], st["x"], st["w"], st["sc"], st["sf"])
    if call == "static":
        L.lrcnn_forward_rows_static(*a, st["y"])
        return dict(y=st["y"])
    if call == "forward":
        L.lrcnn_forward_rows(*a, st["y"], st["ws"])
        return dict(y=st["y"])
    if call == "layerwise":
        L.lrcnn_layerwise_reference_gpu(*a, st["dy"], st["y"], st["dw"], st["dx"], st["ws"])
    else:
        L.lrcnn_forward_rows(*a, st["y"], st["ws"])
        L.lrcnn_backward_rows(*a, st["dy"], st["dw"], st["dx"], st["ws"])
    out = dict(y=st["y"], dw=[d for d in st["dw"] if d is not None])
    if st["dx"] is not None:
        out["dx"] = st["dx"]
    return out


def work(case):
    nodes = _nodes(case)
    ch, size = _channels(nodes, case["c"]), _sizes(nodes, case["h"], case["w"])
    es = 2 if case["bf16"] else 4
    b = case["batch"]
    x = b * case["h"] * case["w"] * case["c"]
    y = b * size[-1][0] * size[-1][1] * ch[-1]
    back = case["call"] in ("step", "layerwise", "train")
    weights, flops = 0, 0.0
    for v, nd in enumerate(nodes[1:], start=1):
        if nd[0] != CONV:
            continue
        k = nd[4] * nd[5] * ch[nd[1]]
        f = 2.0 * b * size[v][0] * size[v][1] * k * nd[3]
        weights += nd[3] * k
        # forward; weight gradient; input gradient (of the input itself only
        # where it is asked for)
        flops += f * (1 + (2 if nd[1] or case["dx"] else 1) * back)
    total = es * (x + y + weights)
    if back:
        total += 4 * weights + es * y * (case["call"] != "train") + es * x * case["dx"]
    if case["call"] == "train":
        k = y // b
        flops += 6.0 * b * k * CLASSES
        total += 4 * (weights + 3 * CLASSES * k)
    return {"bytes": float(total), "flops": flops}


def tolerance(case):
    # Four times what the same passes show when every convolution sums its K
    # products in another order (wider K steps, other split counts). A sum
    # that lands on the other side of zero switches a ReLU, so gradients
    # differ by far more than the sums themselves (about the root of the
    # share of switched sites), most through a whole network and in bfloat16.
    # Seen: float32 blocks 1.5e-3 (largest single value 0.4);
    # VGG-16 1.4e-2; bfloat16 blocks 4.6e-3 (0.3); ResNet-50's output 8e-3.
    if case["net"] in ("vgg16", "resnet50"):
        return {"rel": 0.03, "max": 0.99}
    return {"rel": 0.02 if case["bf16"] else 0.006, "max": 0.99}


def _conv(x, w, nd):
    """One image [H][W][C] in float64."""
    (_op, _i, _j, _c, kh, kw, sh, sw, ph, pw, _a, _r) = nd
    xp = torch.nn.functional.pad(x, (0, 0, pw, pw, ph, ph))
    ho, wo = (xp.shape[0] - kh) // sh + 1, (xp.shape[1] - kw) // sw + 1
    out = torch.zeros((ho * wo, w.shape[0]), dtype=x.dtype, device=x.device)
    for i in range(kh):
        for j in range(kw):
            t = xp[i:i + (ho - 1) * sh + 1:sh, j:j + (wo - 1) * sw + 1:sw].reshape(ho * wo, -1)
            out.addmm_(t, w[:, i, j, :].t().contiguous())
    return out.view(ho, wo, -1)


def _conv_back(x, w, nd, g, want_x):
    (_op, _i, _j, _c, kh, kw, sh, sw, ph, pw, _a, _r) = nd
    xp = torch.nn.functional.pad(x, (0, 0, pw, pw, ph, ph))
    ho, wo = g.shape[:2]
    gf = g.reshape(ho * wo, -1)
    gt = gf.t().contiguous()
    dw = torch.empty_like(w)
    dxp = torch.zeros_like(xp) if want_x else None
    for i in range(kh):
        for j in range(kw):
            at = (slice(i, i + (ho - 1) * sh + 1, sh), slice(j, j + (wo - 1) * sw + 1, sw))
            dw[:, i, j, :] = gt @ xp[at].reshape(ho * wo, -1)
            if want_x:
                dxp[at] += (gf @ w[:, i, j, :].contiguous()).view(ho, wo, -1)
    if not want_x:
        return dw, None
    return dw, dxp[ph:ph + x.shape[0], pw:pw + x.shape[1]]


def _pool(x, nd):
    (_op, _i, _j, _c, kh, kw, sh, sw, ph, pw, _a, _r) = nd
    xp = torch.nn.functional.pad(x, (0, 0, pw, pw, ph, ph), value=-math.inf)
    ho, wo = (xp.shape[0] - kh) // sh + 1, (xp.shape[1] - kw) // sw + 1
    best, arg = None, None
    for i in range(kh):
        for j in range(kw):
            t = xp[i:i + (ho - 1) * sh + 1:sh, j:j + (wo - 1) * sw + 1:sw]
            if best is None:
                best, arg = t.clone(), torch.zeros(t.shape, dtype=torch.uint8, device=t.device)
            else:
                up = t > best
                best = torch.where(up, t, best)
                arg[up] = i * kw + j
    return best, arg


def _pool_back(x, nd, arg, g):
    (_op, _i, _j, _c, kh, kw, sh, sw, ph, pw, _a, _r) = nd
    ho, wo = g.shape[:2]
    dxp = torch.zeros((x.shape[0] + 2 * ph, x.shape[1] + 2 * pw, x.shape[2]), dtype=x.dtype,
                      device=x.device)
    for i in range(kh):
        for j in range(kw):
            dxp[i:i + (ho - 1) * sh + 1:sh, j:j + (wo - 1) * sw + 1:sw] += g * (arg == i * kw + j)
    return dxp[ph:ph + x.shape[0], pw:pw + x.shape[1]]


def _image(nodes, x, ws, scs, sfs, dy, want_dx, dws):
    """Output and (dy given) gradients of one image in float64; the weight
    gradients are added to dws. dy may be a function of the output."""
    maps, args = [x], [None]
    for v, nd in enumerate(nodes[1:], start=1):
        arg = None
        if nd[0] == CONV:
            z = _conv(maps[nd[1]], ws[v], nd)
            if nd[10]:
                z = z * scs[v] + sfs[v]
        elif nd[0] == POOL:
            z, arg = _pool(maps[nd[1]], nd)
        else:
            z = maps[nd[1]] + maps[nd[2]]
        maps.append(z.clamp_(min=0) if nd[11] else z)
        args.append(arg)
    y = maps[-1]
    if dy is None:
        return y, None
    err = [None] * len(nodes)
    err[-1] = dy(y) if callable(dy) else dy

    def add(u, e):
        err[u] = e if err[u] is None else err[u] + e

    for v in range(len(nodes) - 1, 0, -1):
        nd, g = nodes[v], err[v]
        err[v] = None
        if nd[11]:
            g = g * (maps[v] > 0)
        if nd[0] == CONV:
            g = g * scs[v] if nd[10] else g
            want = nd[1] > 0 or want_dx
            dw, e = _conv_back(maps[nd[1]], ws[v], nd, g, want)
            dws[v] += dw
            if want:
                add(nd[1], e)
        elif nd[0] == POOL:
            add(nd[1], _pool_back(maps[nd[1]], nd, args[v], g))
        else:
            add(nd[1], g)
            add(nd[2], g)
        maps[v] = None
    return y, err[0] if want_dx else None


def exact(case, seed):
    nodes, x, ws, scs, sfs, dy = _inputs(case, seed)

    def wide(ts):
        return [None if t is None else t.double() for t in ts]

    ws, scs, sfs = wide(ws), wide(scs), wide(sfs)
    dws = [None if w is None else torch.zeros_like(w) for w in ws]
    back = case["call"] in ("step", "layerwise", "train")
    train = case["call"] == "train"
    ys, dxs, logits, losses = [], [], [], []
    if train:
        fc_w, fc_b, labels = _head_inputs(nodes, case, seed)
        fc_w, fc_b = fc_w.double(), fc_b.double()
        d_fc_w, d_fc_b = torch.zeros_like(fc_w), torch.zeros_like(fc_b)
    for b in range(case["batch"]):
        up = None
        if train:
            def up(y, b=b):
                z = fc_w @ y.reshape(-1) + fc_b
                logits.append(z)
                losses.append(torch.logsumexp(z, 0) - z[labels[b].long()])
                d = torch.softmax(z, 0)
                d[labels[b].long()] -= 1
                d /= case["batch"]
                d_fc_w.add_(torch.outer(d, y.reshape(-1)))
                d_fc_b.add_(d)
                return (fc_w.t().contiguous() @ d).view(y.shape)
        elif back:
            up = dy[b].double()
        y, dx = _image(nodes, x[b].double(), ws, scs, sfs, up, case["dx"], dws)
        ys.append(y)
        dxs.append(dx)
    dw = [d for d in dws if d is not None]
    if train:
        return dict(loss=torch.stack(losses).mean(), logits=torch.stack(logits),
                    w=[w - LR * d for w, d in zip(ws, dws) if w is not None], dw=dw,
                    fc_w=fc_w - LR * d_fc_w, fc_b=fc_b - LR * d_fc_b, d_fc_w=d_fc_w,
                    d_fc_b=d_fc_b)
    out = dict(y=torch.stack(ys))
    if back:
        out["dw"] = dw
        if case["dx"]:
            out["dx"] = torch.stack(dxs)
    return out
