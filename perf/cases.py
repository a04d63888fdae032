"""The work whose speed counts, as cases: what HetPipe's virtual workers do all day.

A virtual worker runs the training step of its pipeline stage (hp.Stage: forward and
backward of a list of layers) for every minibatch and the WSP update of its weights
(hp.ParameterServer, hp.VirtualWorker) after it.  The stages are runs of layers of VGG-19
and ResNet-152 with ImageNet-sized inputs at batch 32 in fp32 or bf16, the Tiny CNN is the
smallest network, and partitions are cut at any layer, so single convolutions, blocks and
heads are stages of their own.

A case is a dict of plain values; `kind` says which layers it has:
  conv   one convolution (optionally ReLU, then 2x2 max-pool) of the VGG kind
  image  VGG's first block: two 3x3 convolutions with ReLU on an image, max-pool; no
         gradient of the image
  block  a ResNet bottleneck (1x1, 3x3, 1x1, batch norms, residual add)
  stem   ResNet's 7x7/2 convolution on an image, batch norm, ReLU, 3x3/2 max-pool
  head   three fully connected layers and the loss
  vgg19  the whole network: logits, loss and every weight gradient
  tiny   a wave of the Tiny CNN's virtual workers through the driver
  wave   the WSP update alone: a wave of local updates and its fused end
"""
import math

import torch
import torch.nn.functional as F

from paper_2005_14038_amd import hetpipe as hp
from paper_2005_14038_amd import nets
from paper_2005_14038_amd.driver import WSPDriver

LR = 0.01


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest calls: 16x16 images, batch 4, two workers of waves of four; launches
        # and the host's work decide
        dict(name="tiny_wave", kind="tiny", dtype="fp32", batch=4, h=16, w=16, vws=2, W=4),
        # the weight update of a worker that holds the whole VGG-19 (143.7 M parameters)
        dict(name="wsp_wave_vgg19", kind="wave", dtype="fp32", params=143667240, W=4),
        # VGG-19's classifier, the last stage of its pipeline
        dict(name="head_fp32", kind="head", dtype="fp32", batch=32, h=7, w=7, c=512, width=4096,
             classes=1000),
        # VGG-19's first block on 224x224 images, the start of its first stage
        dict(name="image_block_fp32", kind="image", dtype="fp32", batch=32, h=224, w=224, c=3,
             k=64),
        # conv3_2 of VGG-19: the layer most of the first stage's time goes to
        dict(name="conv56_fp32", kind="conv", dtype="fp32", batch=32, h=56, w=56, c=256, k=256,
             r=3, stride=1, pad=1, relu=True, pool=False),
        # sizes that fit no tile: a partial batch, odd maps, channel counts of a pruned net
        dict(name="conv_ragged_fp32", kind="conv", dtype="fp32", batch=6, h=29, w=35, c=200,
             k=136, r=3, stride=1, pad=1, relu=False, pool=False),
        # conv4_x of ResNet-152 (36 of its 50 blocks), fp32 as in the middle-stage benchmark
        dict(name="block14_fp32", kind="block", dtype="fp32", batch=32, h=14, w=14, c=1024,
             mid=256, stride=1, project=False),
        # the block that starts the middle stage: projection shortcut, stride 2
        dict(name="block56_down_fp32", kind="block", dtype="fp32", batch=32, h=56, w=56, c=256,
             mid=128, stride=2, project=True),
        # the same conv4_x block in bf16, as the ResNet-152 workload runs it
        dict(name="block14_bf16", kind="block", dtype="bf16", batch=32, h=14, w=14, c=1024,
             mid=256, stride=1, project=False),
        # ResNet-152's stem in bf16
        dict(name="stem_bf16", kind="stem", dtype="bf16", batch=32, h=224, w=224, c=3, k=64),
        # conv4_2 of VGG-19 in bf16
        dict(name="conv28_bf16", kind="conv", dtype="bf16", batch=32, h=28, w=28, c=512, k=512,
             r=3, stride=1, pad=1, relu=True, pool=False),
        # the headline step: VGG-19 at batch 32 in fp32, forward and backward
        dict(name="vgg19_fp32", kind="vgg19", dtype="fp32", batch=32, h=224, w=224, width=4096,
             classes=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: batches 1 to 32, maps from the images' 224 down to 7, channel counts of
    the two networks (8 to 2048 with the map) or any between, both data types."""
    kind = rng.choice(["conv"] * 4 + ["block"] * 4 + ["head", "image", "stem", "tiny", "wave",
                                                      "vgg19"])
    dtype = rng.choice(["fp32", "fp32", "bf16"])
    batch = rng.choice([32, 32, _log(rng, 1, 32)])
    odd = rng.random() < 0.4
    if kind == "conv":
        h = rng.choice([14, 28, 56, 112])
        top = {14: 512, 28: 512, 56: 256, 112: 128}[h]
        c, k = rng.choice([top // 2, top]), top
        if odd:
            h, c, k = rng.randint(7, h), rng.randint(8, top), rng.randint(8, top)
        w = h + (rng.randint(-3, 9) if odd else 0)
        r = rng.choice([3, 3, 1])
        return dict(kind=kind, dtype=dtype, batch=batch, h=h, w=w, c=c, k=k, r=r,
                    stride=rng.choice([1, 1, 1, 2]), pad=r // 2, relu=rng.random() < 0.7,
                    pool=False)
    if kind == "block":
        h = rng.choice([14, 28, 56])
        mid = {14: 256, 28: 128, 56: 64}[h]
        project = rng.random() < 0.3
        w = h
        if odd:
            h, w, mid = rng.randint(7, h), rng.randint(7, h), rng.randint(4, mid // 4) * 4
        return dict(kind=kind, dtype=dtype, batch=max(2, batch), h=h, w=w, c=4 * mid,
                    mid=2 * mid if project else mid, stride=2 if project else 1, project=project)
    if kind == "head":
        return dict(kind=kind, dtype=dtype, batch=batch, h=7, w=7, c=_log(rng, 32, 512),
                    width=4 * _log(rng, 64, 1024), classes=_log(rng, 10, 1000))
    if kind == "image":
        h = rng.randint(16, 112) * 2
        return dict(kind=kind, dtype=dtype, batch=batch, h=h, w=h, c=3, k=64)
    if kind == "stem":
        h = rng.randint(32, 224)
        return dict(kind=kind, dtype=dtype, batch=max(2, batch), h=h, w=h, c=3, k=64)
    if kind == "tiny":
        return dict(kind=kind, dtype="fp32", batch=rng.randint(1, 16), h=2 * rng.randint(4, 16),
                    w=2 * rng.randint(4, 16), vws=rng.randint(1, 4), W=rng.randint(1, 6))
    if kind == "wave":
        return dict(kind=kind, dtype="fp32", params=_log(rng, 10_000, 143_667_240),
                    W=rng.randint(1, 6))
    # fp32: in bf16 the gradients of so deep a network are not determined to a few per cent
    return dict(kind=kind, dtype="fp32", batch=_log(rng, 2, 31), h=32 * rng.randint(2, 6),
                w=32 * rng.randint(2, 6), width=_log(rng, 256, 4096), classes=_log(rng, 10, 1000))


# ------------------------------------------------------------------ the stages
def _builder(case):
    kind, h, w = case["kind"], case["h"], case["w"]
    if kind == "tiny":
        return nets.tiny(h, w)
    if kind == "vgg19":
        return nets.vgg19(h, w, classes=case["classes"], width=case["width"])
    b = nets.Builder(h, w, case["c"])
    if kind == "conv":
        x = b.conv(-1, case["k"], case["r"], case["stride"], case["pad"], bias=True)
        if case["relu"]:
            x = b.relu(x)
        if case["pool"]:
            b.maxpool(x, 2, 2)
    elif kind == "image":
        x = b.relu(b.conv(-1, case["k"], 3, 1, 1, bias=True))
        x = b.relu(b.conv(x, case["k"], 3, 1, 1, bias=True))
        b.maxpool(x, 2, 2)
    elif kind == "block":
        # up to the residual add: the partition is cut before the block's last ReLU, whose
        # mask would pass single gradients straight into dx, where a pre-activation within
        # round-off of zero decides a whole element
        mid, stride = case["mid"], case["stride"]
        y = b.relu(b.bn(b.conv(-1, mid, 1)))
        y = b.relu(b.bn(b.conv(y, mid, 3, stride, 1)))
        y = b.bn(b.conv(y, 4 * mid, 1))
        b.add(y, b.bn(b.conv(-1, 4 * mid, 1, stride)) if case["project"] else -1)
    elif kind == "stem":
        x = b.relu(b.bn(b.conv(-1, case["k"], 7, 2, 3)))
        b.maxpool(x, 3, 2, 1)
    elif kind == "head":
        x = b.relu(b.fc(-1, case["width"]))
        x = b.relu(b.fc(x, case["width"]))
        b.ce(b.fc(x, case["classes"]))
    return b


IMAGE = ("image", "stem", "vgg19", "tiny")   # these read images; a first stage asks for no dx


def _weights(layers, gen):
    """He-normal weights, small biases, batch norms near the identity, as one flat vector."""
    parts = []

    def normal(n, std, mean=0.0):
        parts.append(torch.randn(n, device="cuda", generator=gen) * std + mean)

    for d in layers:
        if d["kind"] in (hp.HP_CONV, hp.HP_FC):
            fan = d["C"] * (d["R"] * d["S"] if d["kind"] == hp.HP_CONV else 1)
            normal(d["K"] * fan, math.sqrt(2.0 / fan))
            if d.get("bias"):
                normal(d["K"], 0.01)
        elif d["kind"] == hp.HP_BN:
            normal(d["C"], 0.1, 1.0)
            normal(d["C"], 0.1)
    return torch.cat(parts)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _data(case, b, seed):
    """Weights, one minibatch's input (an image, or the ReLU output of the layer before),
    labels or the gradient that the next stage sends."""
    gen = _gen(seed)
    w = _weights(b.layers, gen)
    h, wd, c = b.input_shape
    x = torch.randn(case["batch"], h, wd, c, device="cuda", generator=gen)
    if case["kind"] not in IMAGE:
        x = x.relu_()
    labels = dy = None
    if b.layers[-1]["kind"] == hp.HP_SOFTMAX_CE:
        classes = b.layers[-1]["K"]
        labels = torch.randint(0, classes, (case["batch"],), device="cuda", generator=gen,
                               dtype=torch.int32)
    else:
        shape = (case["batch"],) + tuple(b.shape[len(b.layers) - 1])
        dy = torch.randn(shape, device="cuda", generator=gen) * 1e-3
    return w, x, labels, dy


class _Memory:
    """A device buffer of the library, for torch.as_tensor; keeps the object that owns it."""

    def __init__(self, owner, ptr, n):
        self.owner = owner
        self.__cuda_array_interface__ = dict(shape=(n,), typestr="<f4", data=(ptr, False),
                                             version=2, strides=None)


def _view(owner, ptr, n):
    t = torch.as_tensor(_Memory(owner, ptr, n), device="cuda")
    t.owner = owner
    return t


def prepare(case, seed):
    kind = case["kind"]
    stream = torch.cuda.current_stream()
    if kind == "wave":
        gen = _gen(seed)
        P, W = case["params"], case["W"]
        w0 = torch.randn(P, device="cuda", generator=gen) * 0.02
        grads = [torch.randn(P, device="cuda", generator=gen) * 1e-3 for _ in range(W)]
        ps = hp.ParameterServer(P, w0, 1, 0, stream)
        vw = hp.VirtualWorker(ps, 0, W - 1)
        ring, stride, ut = vw.buffers()
        views = dict(wg=_view(vw, ps.weights_ptr(), P), ut=_view(vw, ut, P),
                     ring=[_view(vw, ring + 4 * s * stride, P) for s in range(W)])
        return dict(case=case, vw=vw, ps=ps, grads=grads, views=views)
    b = _builder(case)
    h, wd, c = b.input_shape
    st = hp.Stage(b.layers, case["batch"], h, wd, c, dtype=case["dtype"], stream=stream)
    if kind == "tiny":
        w0 = _data(case, b, seed)[0]
        data = [_data(case, b, seed + 1 + i) for i in range(case["vws"] * case["W"])]

        def minibatch(n, q):
            d = data[n * case["W"] + (q - 1) % case["W"]]
            return d[1], d[2], None

        drv = WSPDriver(st, w0, case["vws"], case["W"] - 1, 0, LR, minibatch, stream=stream)
        uts = [_view(v, v.buffers()[2], st.P) for v in drv.vws]
        return dict(case=case, drv=drv, stage=st, waves=0, uts=uts,
                    wg=_view(drv.ps, drv.ps.weights_ptr(), st.P), data=data)
    w, x, labels, dy = _data(case, b, seed)
    H, W_, C = st.output_shape(-1)
    out = dict(y=torch.empty((case["batch"], H, W_, C), device="cuda"),
               grad=torch.empty(st.P, device="cuda"))
    if labels is not None:
        out["loss"] = torch.empty(1, device="cuda")
    if kind not in IMAGE:
        out["dx"] = torch.empty_like(x)
    return dict(case=case, stage=st, w=w, x=x, labels=labels, dy=dy, out=out)


def run(state):
    kind = state["case"]["kind"]
    if kind == "wave":
        vw, grads = state["vw"], state["grads"]
        for i, g in enumerate(grads):
            vw.weights()
            if i + 1 < len(grads):
                vw.local_update(g, LR)
            else:
                vw.wave_end(g, LR)
        return state["views"]
    if kind == "tiny":
        drv = state["drv"]
        state["waves"] += 1
        drv.run(state["waves"])
        return dict(wg=state["wg"], uts=state["uts"], y=drv.y, loss=drv.loss, grad=drv.grad)
    st, out = state["stage"], state["out"]
    st.forward(state["w"], state["x"], out["y"], state["labels"], out.get("loss"))
    st.backward(state["w"], state["dy"], out.get("dx"), out["grad"])
    return out


# ------------------------------------------------------------------ work and tolerances
def work(case):
    kind = case["kind"]
    if kind == "wave":
        # per parameter and call: a local update reads the gradient and the newest version
        # and writes a version and u~ (which all but a wave's first read too); the wave's
        # end reads the gradient, u~ and w_g and writes u~, w_g and the pulled version
        W = case["W"]
        per = 20 if W == 1 else 16 + 20 * (W - 2) + 24
        return dict(bytes=per * case["params"], flops=3 * W * case["params"])
    b = _builder(case)
    flops, params = 0, b.param_count()
    first = True
    for i, d in enumerate(b.layers):
        if d["kind"] in (hp.HP_CONV, hp.HP_FC):
            h, w, k = b.shape[i]
            mac = case["batch"] * h * w * k * d["C"]
            if d["kind"] == hp.HP_CONV:
                mac *= d["R"] * d["S"]
            # forward, weight gradient, and the data gradient where one is asked for
            flops += 2 * mac * (2 if first and kind in IMAGE else 3)
            first = False
    h, w, c = b.input_shape
    x = case["batch"] * h * w * c
    h, w, c = b.shape[len(b.layers) - (2 if b.layers[-1]["kind"] == hp.HP_SOFTMAX_CE else 1)]
    y = case["batch"] * h * w * c
    values = params * 2 + x + y + (0 if kind in IMAGE else x)    # w, grad, x, y, dx
    if b.layers[-1]["kind"] != hp.HP_SOFTMAX_CE:
        values += y                                              # dy
    if kind == "tiny":
        steps = case["vws"] * case["W"]
        return dict(bytes=4 * steps * (values + 4 * params), flops=steps * flops)
    return dict(bytes=4 * values, flops=flops)


def tolerance(case):
    """About four times what the path is off its 64-bit value.  Sums in 32 bits stay below
    1e-6; where a ReLU or a pool lies on the path, the few pre-activations within round-off
    of zero (of a tie) go either way, and every one moves the gradients by a whole term."""
    kind = case["kind"]
    if kind == "wave":
        return "exact"            # one rounding per operation, in the order of the definition
    if kind == "tiny":
        return dict(rel=1e-3, max=0.5)
    if case["dtype"] == "bf16":   # rounding ties of the operands as well: 4e-3 in a block
        return dict(rel=2e-2, max=0.9)
    if kind == "conv" and not case["relu"]:
        return dict(rel=2e-6, max=1e-4)
    if kind == "conv":            # 1e-4
        return dict(rel=5e-4 if case["batch"] * case["h"] * case["w"] > 50000 else 5e-3, max=0.9)
    return dict(rel=5e-3, max=0.9)  # 4e-4 to 9e-4


# ------------------------------------------------------------------ 64-bit results
class _Conv(torch.autograd.Function):
    """A convolution (NHWC, weights [K][R][S][C]) tap by tap as matrix products in 64 bits;
    in bf16 mode every operand is first rounded to bf16, which is what that mode means."""

    @staticmethod
    def forward(ctx, x, w, stride, pad, low):
        rnd = (lambda t: t.float().bfloat16().double()) if low else (lambda t: t)
        xr, wr = rnd(x), rnd(w)
        ctx.save_for_backward(xr, wr)
        ctx.args = (stride, pad, rnd)
        N, H, W, C = x.shape
        K, R, S, _ = w.shape
        P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
        ctx.pq = P, Q
        xp = F.pad(xr, (0, 0, pad, pad, pad, pad))
        y = torch.zeros(N * P * Q, K, dtype=x.dtype, device=x.device)
        for r in range(R):
            for s in range(S):
                xs = xp[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride]
                y += xs.reshape(-1, C) @ wr[:, r, s].t().contiguous()
        return y.view(N, P, Q, K)

    @staticmethod
    def backward(ctx, dy):
        xr, wr = ctx.saved_tensors
        stride, pad, rnd = ctx.args
        P, Q = ctx.pq
        N, H, W, C = xr.shape
        K, R, S, _ = wr.shape
        d = rnd(dy).reshape(-1, K)
        dt = d.t().contiguous()
        xp = F.pad(xr, (0, 0, pad, pad, pad, pad))
        dxp = torch.zeros_like(xp)
        dw = torch.empty_like(wr)
        for r in range(R):
            for s in range(S):
                at = (slice(None), slice(r, r + stride * (P - 1) + 1, stride),
                      slice(s, s + stride * (Q - 1) + 1, stride))
                dw[:, r, s] = dt @ xp[at].reshape(-1, C)
                dxp[at] += (d @ wr[:, r, s].contiguous()).view(N, P, Q, C)
        return dxp[:, pad:pad + H, pad:pad + W], dw, None, None, None


def _graph(layers, flat, x, labels, low):
    """The stage's output and, with labels, its loss."""
    vals, at = {-1: x}, 0

    def take(*shape):
        nonlocal at
        n = math.prod(shape)
        at += n
        return flat[at - n:at].view(shape)

    for i, d in enumerate(layers):
        v, k = vals[d.get("in0", i - 1)], d["kind"]
        if k in (hp.HP_CONV, hp.HP_FC):
            r = d["R"] if k == hp.HP_CONV else 1
            if k == hp.HP_FC:
                v = v.reshape(v.shape[0], 1, 1, -1)
            w = take(d["K"], r, r, d["C"])
            v = _Conv.apply(v, w, d.get("stride", 1), d.get("pad", 0), low)
            if d.get("bias"):
                v = v + take(d["K"])
        elif k == hp.HP_RELU:
            v = v.relu()
        elif k == hp.HP_MAXPOOL:
            v = F.max_pool2d(v.permute(0, 3, 1, 2), d["R"], d["stride"], d["pad"])
            v = v.permute(0, 2, 3, 1)
        elif k == hp.HP_BN:
            gamma, beta = take(d["C"]), take(d["C"])
            mean = v.mean((0, 1, 2))
            var = (v - mean).square().mean((0, 1, 2))
            v = (v - mean) / (var + d["eps"]).sqrt() * gamma + beta
        elif k == hp.HP_ADD:
            v = v + vals[d["in1"]]
        elif k == hp.HP_SOFTMAX_CE:
            z = v.reshape(v.shape[0], -1)
            return v, F.cross_entropy(z, labels.long())
        vals[i] = v
    return vals[len(layers) - 1], None


def _step64(case, b, w, x, labels, dy):
    w = w.double().requires_grad_()
    x = x.double().requires_grad_(case["kind"] not in IMAGE)
    y, loss = _graph(b.layers, w, x, labels, case["dtype"] == "bf16")
    if loss is not None:
        loss.backward()
    else:
        y.backward(dy.double())
    return y.detach(), loss, w.grad, x.grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "wave":
        gen = _gen(seed)
        P, W = case["params"], case["W"]
        w = (torch.randn(P, device="cuda", generator=gen) * 0.02).double()
        ut = torch.zeros_like(w)
        ring = []
        for _ in range(W):
            u = -LR * (torch.randn(P, device="cuda", generator=gen) * 1e-3).double()
            ut += u
            w = w + u
            ring.append(w)
        return dict(wg=w, ut=ut, ring=ring)
    b = _builder(case)
    if kind == "tiny":
        # every minibatch of the first wave reads the initial weights
        w0 = _data(case, b, seed)[0]
        uts = []
        for n in range(case["vws"]):
            ut = torch.zeros_like(w0, dtype=torch.float64)
            for q in range(case["W"]):
                _, x, labels, _ = _data(case, b, seed + 1 + n * case["W"] + q)
                y, loss, grad, _ = _step64(case, b, w0, x, labels, None)
                ut -= LR * grad
            uts.append(ut)
        return dict(wg=w0.double() + sum(uts), uts=uts, y=y, loss=loss.detach().view(1),
                    grad=grad)
    w, x, labels, dy = _data(case, b, seed)
    y, loss, grad, dx = _step64(case, b, w, x, labels, dy)
    out = dict(y=y, grad=grad)
    if loss is not None:
        out["loss"] = loss.detach().view(1)
    if dx is not None:
        out["dx"] = dx
    return out
