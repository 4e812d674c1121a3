"""The work this framework is measured on: forward, recomputation and backward of the networks its
benchmark configurations name (bottleneck stacks, whole ResNet-50, a BERT-base encoder layer, the
operator-granular batch-norm chain), each through the C ABI's binding as a training program drives it.

A case is one stage of such a program: its tensors live in the library's arena, descriptors and
data-gradient weights are laid out once, and a pass is the calls of one iteration.  Activations that
a backward pass reads are inputs of the case (what an earlier forward pass stored), so that its ReLU
masks are given.  "both" is one micro-batch's forward and the backward of the micro-batch before it.
Offload and Reload are not here: their time is the copy engines' and the host link's alone.
"""
import math

import torch

import paper_2203_15980_amd as dl
import synth
from paper_2203_15980_amd.harness import find_blocks

DEV = "cuda:0"
EPS = 1e-5
SYNC_EVERY = 16      # passes between two delta_sync calls: a program syncs where it reads its loss; events are recycled there

STAGES = {2: (64, 256), 3: (128, 512), 4: (256, 1024), 5: (512, 2048)}     # stage -> (middle, output) channels


def listed():
    return [
        # configuration 1: three fp32 bottlenecks on 2 x 32 x 32; the smallest calls, launches and latency
        dict(name="f32_stack_b2_32", kind="blocks", do="both", dtype="f32", stage=2, entry=True, blocks=3, N=2, H=32, W=32),
        # configuration 2: conv2_x at batch 32, forward, then every block-internal tensor released and regenerated
        dict(name="conv2x_recompute_b32_56", kind="blocks", do="forward", dtype="bf16", stage=2, entry=True, blocks=3, N=32, H=56, W=56),
        # configuration 2's backward pass
        dict(name="conv2x_backward_b32_56", kind="blocks", do="backward", dtype="bf16", stage=2, entry=True, blocks=3, N=32, H=56, W=56),
        # configuration 3: the strided block that opens conv3_x, with its projection shortcut, at the headline batch
        dict(name="conv3_entry_backward_b128_56", kind="blocks", do="backward", dtype="bf16", stage=3, entry=True, blocks=1, N=128, H=56, W=56),
        # configuration 4 (ResNet-101 at batch 256): an identity block of the last stage
        dict(name="conv5_backward_b256_7", kind="blocks", do="backward", dtype="bf16", stage=5, entry=False, blocks=1, N=256, H=7, W=7),
        # a few images of an odd size through a late block: too little work to fill the chip, ragged tiles
        dict(name="conv4_b3_13x17", kind="blocks", do="both", dtype="bf16", stage=4, entry=False, blocks=1, N=3, H=13, W=17),
        # configuration 3's whole forward pass with the loss
        dict(name="resnet50_forward_b128_224", kind="resnet", N=128, image=224),
        # the tail of its backward pass: max-pool with the stem's ReLU mask, then the stem's weight gradient
        dict(name="stem_backward_b128_224", kind="stem", N=128, image=224),
        # its top: average pool, classifier, loss, and their backward
        dict(name="head_b128", kind="head", N=128, H=7, W=7),
        # configuration 5: one encoder layer at 32 x 512 tokens
        dict(name="encoder_b32_512", kind="encoder", N=32, S=512),
        # the same layer on one short odd sequence, as a serving program calls it
        dict(name="encoder_b1_77", kind="encoder", N=1, S=77),
        # operator granularity (batch statistics): batch-norm, residual add, ReLU and back, at conv3_x's output size
        dict(name="bn_add_relu_b32_28", kind="bn", N=32, H=28, W=28, C=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["blocks"] * 6 + ["resnet", "stem", "head", "encoder", "encoder", "bn"])
    if kind == "blocks":
        f32 = rng.random() < 0.15
        stage = 2 if f32 else rng.choice([2, 3, 4, 5])
        entry = rng.random() < 0.4
        side = {2: 56, 3: 28, 4: 14, 5: 7}[stage] * (2 if entry and stage > 2 else 1)
        lo = max(5, side // 2)
        H, W = rng.randint(lo, side), rng.randint(lo, side)
        most = 2 if f32 else {2: 32, 3: 128, 4: 128, 5: 256}[stage]
        return dict(kind="blocks", do=rng.choice(["forward", "backward", "both"]), dtype="f32" if f32 else "bf16", stage=stage,
                    entry=entry, blocks=3 if stage == 2 and entry else 1, N=_log(rng, 1, most), H=H if not f32 else min(H, 32),
                    W=W if not f32 else min(W, 32))
    if kind == "resnet":
        return dict(kind="resnet", N=_log(rng, 1, 128), image=rng.choice([160, 192, 224]) + rng.choice([0, 0, -3, -1]))
    if kind == "stem":
        return dict(kind="stem", N=_log(rng, 1, 128), image=rng.choice([96, 160, 192, 224]) + rng.choice([0, 0, -3, -1]))
    if kind == "head":
        return dict(kind="head", N=_log(rng, 1, 256), H=rng.randint(3, 8), W=rng.randint(3, 8))
    if kind == "encoder":
        return dict(kind="encoder", N=_log(rng, 1, 32), S=rng.randint(17, 512))
    return dict(kind="bn", N=_log(rng, 1, 32), H=rng.randint(7, 56), W=rng.randint(7, 56), C=rng.choice([64, 128, 256, 512]))


# ------------------------------------------------------------------ networks and inputs

def _layers(case):
    k = case["kind"]
    if k == "blocks":
        mid, cout = STAGES[case["stage"]]
        cin = {2: 64}.get(case["stage"], mid * 2) if case["entry"] else cout
        layers, x, H, W = [], "x0", case["H"], case["W"]
        for b in range(case["blocks"]):
            first = case["entry"] and b == 0
            stride = 2 if first and case["stage"] > 2 else 1
            p, Ho, Wo = "b%d" % (b + 1), (H - 1) // stride + 1, (W - 1) // stride + 1
            spec = lambda n, xin, res, h, w, ci, co, R, s, relu: layers.append(synth.LayerSpec(      # noqa: E731
                p + n, "conv", xin, res, p + n, case["N"], h, w, ci, co, R, R, s, R // 2, relu))
            spec(".a1", x, None, H, W, cin, mid, 1, 1, True)
            spec(".a2", p + ".a1", None, H, W, mid, mid, 3, stride, True)
            if first:
                spec(".sc", x, None, H, W, cin, cout, 1, stride, False)
            spec(".out", p + ".a2", p + ".sc" if first else x, Ho, Wo, mid, cout, 1, 1, True)
            x, H, W, cin = p + ".out", Ho, Wo, cout
        return layers
    if k == "resnet":
        return synth.resnet_layers(case["N"], (3, 4, 6, 3), image=case["image"])
    if k == "stem":
        return synth.resnet_layers(case["N"], (3, 4, 6, 3), image=case["image"])[:2]
    if k == "head":
        N, H, W = case["N"], case["H"], case["W"]
        return [synth.LayerSpec("avgpool", "avgpool", "x0", None, "avgpool", N, H, W, 2048, 2048, H, W, 1, 0, False),
                synth.LayerSpec("fc", "fc", "avgpool", None, "logits", N, 1, 1, 2048, 1000, 1, 1, 1, 0, False)]
    if k == "encoder":
        return synth.encoder_layers(case["N"], case["S"], nlayers=1)
    return []


def _tdtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _inputs(case, seed):
    """Every input and parameter of a case, from the seed alone: name -> GPU tensor."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    t = _tdtype(case)
    rn = lambda *s: torch.randn(*s, device=DEV, generator=g)                       # noqa: E731
    un = lambda lo, hi, n: lo + (hi - lo) * torch.rand(n, device=DEV, generator=g)  # noqa: E731
    v, k = {}, case["kind"]
    if k == "bn":
        shape = (case["N"], case["H"], case["W"], case["C"])
        C = case["C"]
        v["x"] = (rn(*shape) * un(0.5, 1.5, C) + 0.3 * rn(C)).to(t)                # a convolution's output, per-channel mean and spread
        v["res"] = rn(*shape).relu_().to(t)
        v["gy"] = rn(*shape).to(t)
        v["gamma"], v["beta"] = un(0.5, 1.5, C), 0.1 * rn(C)
        return v
    layers = _layers(case)
    first = layers[0]
    x = rn(first.N, first.H, first.W, first.Cin)
    v["x0"] = (x.relu_() if k in ("blocks", "head") else x).to(t)                  # a block's input is a ReLU output
    for l in layers:
        fan = l.R * l.S * l.Cin
        if l.kind == "conv":
            v["w:" + l.name] = (rn(l.Cout, l.R, l.S, l.Cin) * math.sqrt(2.0 / fan)).to(t)
            v["gamma:" + l.name], v["beta:" + l.name] = un(0.5, 1.5, l.Cout), 0.1 * rn(l.Cout)
            v["mean:" + l.name], v["var:" + l.name] = 0.1 * rn(l.Cout), un(0.5, 1.5, l.Cout)
        elif l.kind == "fc":
            v["w:" + l.name], v["bias:" + l.name] = (rn(l.Cout, fan) * math.sqrt(2.0 / fan)).to(t), 0.1 * rn(l.Cout)
        elif l.kind == "linear":
            v["w:" + l.name], v["bias:" + l.name] = (0.02 * rn(l.Cout, l.Cin)).to(t), 0.02 * rn(l.Cout)
        elif l.kind == "layernorm":
            v["gamma:" + l.name], v["beta:" + l.name] = un(0.5, 1.5, l.Cout), 0.1 * rn(l.Cout)
    if k in ("head", "resnet"):
        v["labels"] = torch.randint(0, 1000, (case["N"],), device=DEV, generator=g)
    if k == "stem" or (k == "blocks" and case["do"] != "forward"):                 # what an earlier forward pass stored
        for l in layers:
            if not (k == "blocks" and l.y.endswith(".sc")) and not (k == "stem" and l.kind == "maxpool"):
                v["saved:" + l.y] = rn(l.N, l.P, l.Q, l.Cout).relu_().to(t)
        top = layers[-1]
        v["gy"] = rn(top.N, top.P, top.Q, top.Cout).to(t)
    return v


# ------------------------------------------------------------------ one program

class Program:
    """A context, its arena and its tensor table; outputs are views of the arena."""

    def __init__(self, sizes):
        self.ids = {n: i for i, n in enumerate(sizes)}
        self.meta = sizes
        nb = [torch.Size(s).numel() * torch.empty((), dtype=dt).element_size() for s, dt in sizes.values()]
        room = sum((b + 255) // 256 * 256 for b in nb) + max(nb) + (1 << 20)
        self.arena = torch.empty(room, dtype=torch.uint8, device=DEV)
        self.d = dl.Delta(self.arena, torch.cuda.current_stream().cuda_stream)
        self.d.bind(nb)
        self.views, self.keep, self.passes, self.calls = {}, [], 0, []

    def view(self, name):
        ptr = self.d.tensor_ptr(self.ids[name])
        if self.views.get(name, (0, None))[0] != ptr:
            shape, dt = self.meta[name]
            n = torch.Size(shape).numel() * torch.empty((), dtype=dt).element_size()
            off = ptr - self.arena.data_ptr()
            self.views[name] = (ptr, self.arena[off:off + n].view(dt).reshape(shape))
        return self.views[name][1]

    def put(self, name, value):
        self.d.alloc(self.ids[name])
        self.view(name).copy_(value.reshape(self.meta[name][0]))

    def begin(self):
        self.passes += 1
        if self.passes % SYNC_EVERY == 0:
            self.d.sync()


def _desc(p, l, v, code, x=None, y=None, res=None):
    ptr = lambda n: v[n].data_ptr() if n in v else None                            # noqa: E731
    kind = l.kind
    op = {"maxpool": dl.OP_MAXPOOL, "avgpool": dl.OP_AVGPOOL, "attention": dl.OP_ATTENTION, "layernorm": dl.OP_LAYERNORM}.get(kind, dl.OP_CONV)
    scale = shift = None
    if kind == "conv":
        scale, shift = torch.empty(l.Cout, device=DEV), torch.empty(l.Cout, device=DEV)
        p.d.bn_fold(ptr("gamma:" + l.name), ptr("beta:" + l.name), ptr("mean:" + l.name), ptr("var:" + l.name), EPS, l.Cout,
                    scale.data_ptr(), shift.data_ptr())
    elif kind in ("fc", "linear"):
        scale, shift = torch.ones(l.Cout, device=DEV), v["bias:" + l.name]
    elif kind == "layernorm":
        scale, shift = v["gamma:" + l.name], v["beta:" + l.name]
    p.keep += [scale, shift]
    act = 1 if (l.relu and kind == "conv") else (dl.ACT_GELU if l.act == "gelu" else 0)
    xid, yid, rid = x or l.x, y or l.y, res or l.res
    return dl.LayerDesc(x=p.ids[xid], res=p.ids[rid] if rid else dl.NO_TENSOR, y=p.ids[yid], dtype=code, w=ptr("w:" + l.name),
                        scale=scale.data_ptr() if scale is not None else None, shift=shift.data_ptr() if shift is not None else None,
                        N=l.N, H=l.H, W=l.W, Cin=l.Cin, Cout=l.Cout, R=l.R, S=l.S, stride=l.stride, pad=l.pad, relu=act, op=op,
                        eps=synth.LN_EPS if kind == "layernorm" else 0.0)


def _bwd(p, fwd, gy, gx=None, gpre=None, add=None, mask=0, masked=0, wt=None, gw=None, ws=None):
    i = lambda n: p.ids[n] if n else dl.NO_TENSOR                                  # noqa: E731
    return dl.BwdDesc(fwd=fwd, gy=i(gy), gpre=i(gpre or gy), gx=i(gx), gx_add=i(add), mask_gx=mask, gy_masked=masked,
                      wt=wt.data_ptr() if wt is not None else None, gw=gw.data_ptr() if gw is not None else None,
                      workspace=ws.data_ptr() if ws is not None else None, workspace_bytes=ws.numel() if ws is not None else 0)


def _copy(desc):
    return dl.LayerDesc.from_buffer_copy(desc)


def prepare(case, seed):
    v = _inputs(case, seed)
    t, k = _tdtype(case), case["kind"]
    code = dl.DTYPE_F32 if t == torch.float32 else dl.DTYPE_BF16
    if k == "bn":
        return _prepare_bn(case, v, code)
    layers = _layers(case)
    fwd = k != "stem" and case.get("do") != "backward"
    back = k in ("stem", "head") or case.get("do") in ("backward", "both")
    first = layers[0]
    sizes = {"x0": ((first.N, first.H, first.W, first.Cin), t)}
    for l in layers:
        sizes[l.y] = ((l.N, l.P, l.Q, l.Cout), t)
    if "labels" in v:
        sizes["labels"], sizes["loss"] = ((first.N,), torch.int64), ((1,), torch.float32)
    for n in v:
        if n.startswith("saved:"):
            sizes[n] = (tuple(v[n].shape), t)
    if back:
        top = layers[-1]
        sizes["g:" + top.y] = sizes[top.y]
        if k == "blocks":
            sizes["gp"] = sizes[top.y]
            for l in layers:
                if not l.name.endswith(".sc"):
                    sizes["g:" + l.x + (":in" if l.name.endswith(".a1") else "")] = sizes[l.x]
                else:
                    sizes["g:sc"] = sizes[l.x]
        elif k == "stem":
            sizes["g:stem"] = sizes["stem"]
        else:
            sizes["g:avgpool"], sizes["g:x0"] = sizes["avgpool"], sizes["x0"]
    p = Program(sizes)
    for n in sizes:
        if n in v:
            p.put(n, v[n])
    p.keep.append(v)
    p.case, p.names, p.gw = case, [], {}
    desc = {l.y: _desc(p, l, v, code) for l in layers}
    blocks = find_blocks(layers, "f32" if t == torch.float32 else "bf16")
    p.forward = p.rebuild = p.loss = p.backward = None
    p.evict = []
    if fwd:
        every = [_copy(desc[l.y]) for l in layers]
        for i, l in enumerate(layers):
            if any(l.y == chain[0] for chain in blocks.values()):
                every[i].fuse = dl.FUSE_BLOCK
        p.forward = dl.layer_array(every)
        p.names += [l.y for l in layers] if k != "resnet" else [l.y for l in layers if l.y.endswith(".out")] + ["logits"]
        if "labels" in v:
            p.loss = dl.layer_array([dl.LayerDesc(x=p.ids["logits"], res=p.ids["labels"], y=p.ids["loss"], dtype=code, N=first.N, H=1, W=1,
                                                  Cin=1000, Cout=1, R=1, S=1, stride=1, pad=0, relu=0, op=dl.OP_SOFTMAX_CE)])
            p.names.append("loss")
        if k == "blocks" and case["do"] == "forward":        # the block-internal tensors, released and regenerated
            again = []
            for l in layers:
                d = _copy(desc[l.y])
                fused = [c for c in blocks.values() if l.y in c]
                if l.y.endswith(".out"):
                    if not fused:
                        continue
                    d.fuse = dl.FUSE_NO_STORE
                else:
                    p.evict.append(p.ids[l.y])
                    if fused and fused[0][0] == l.y:
                        d.fuse = dl.FUSE_BLOCK
                again.append(d)
            p.rebuild = dl.layer_array(again)
    if back:
        _prepare_backward(p, case, layers, v, code, desc)
    torch.cuda.synchronize()
    return p


def _prepare_backward(p, case, layers, v, code, desc):
    k, d = case["kind"], p.d
    saved = lambda n: "saved:" + n if "saved:" + n in p.ids else n                 # noqa: E731
    # the backward's own view of a layer: it reads the stored activations
    of = {l.y: _desc(p, l, v, code, x=saved(l.x), y=saved(l.y), res=saved(l.res) if l.res and not l.res.endswith(".sc") else l.res)
          for l in layers} if k != "head" else desc
    ws, wt = 16, {}
    for l in layers:
        if l.kind == "conv":
            ws = max(ws, d.backward_workspace(desc[l.y]))
            p.gw[l.name] = torch.zeros(l.Cout, l.R, l.S, l.Cin, device=DEV)
            if k == "blocks":
                wt[l.name] = torch.empty(l.Cout * l.R * l.S * l.Cin * (4 if code == dl.DTYPE_F32 else 2), dtype=torch.uint8, device=DEV)
                d.bwd_weights(desc[l.y], wt[l.name].data_ptr())
        elif l.kind == "fc":
            p.gw[l.name] = torch.zeros(l.Cout * l.Cin + l.Cout, device=DEV)
    work = torch.empty(2 * ws, dtype=torch.uint8, device=DEV)
    p.keep += [work, wt]
    todo = []
    if k == "stem":
        p.put("g:maxpool", v["gy"])
        p.d.alloc(p.ids["g:stem"])
        todo.append(_bwd(p, of["maxpool"], "g:maxpool", gx="g:stem", mask=1))
        todo.append(_bwd(p, of["stem"], "g:stem", masked=1, gw=p.gw["stem"], ws=work))
        p.names.append("g:stem")
    elif k == "head":
        todo.append(dl.BwdDesc(fwd=p.loss[0], gy=dl.NO_TENSOR, gpre=dl.NO_TENSOR, gx=p.ids["g:logits"], gx_add=dl.NO_TENSOR))
        todo.append(_bwd(p, of["logits"], "g:logits", gx="g:avgpool", gw=p.gw["fc"]))
        todo.append(_bwd(p, of["avgpool"], "g:avgpool", gx="g:x0"))
        p.names += ["g:logits", "g:avgpool", "g:x0"]
    else:
        gy, gpre, masked = "g:" + layers[-1].y, "gp", 0
        p.put(gy, v["gy"])
        by = {l.y: l for l in layers}
        for b in range(case["blocks"], 0, -1):
            q = "b%d" % b
            a1, a2, out = by[q + ".a1"], by[q + ".a2"], by[q + ".out"]
            gin, ga1, ga2 = "g:" + a1.x + ":in", "g:" + a1.y, "g:" + a2.y
            kw = lambda n: dict(wt=wt[n], gw=p.gw[n], ws=work)                     # noqa: E731
            todo.append(_bwd(p, of[out.y], gy, gx=ga2, gpre=gpre, mask=1, masked=masked, **kw(out.name)))
            add = gpre
            if q + ".sc" in by:
                todo.append(_bwd(p, of[q + ".sc"], gpre, gx="g:sc", **kw(q + ".sc")))
                add = "g:sc"
            todo.append(_bwd(p, of[a2.y], ga2, gx=ga1, mask=1, masked=1, **kw(a2.name)))
            todo.append(_bwd(p, of[a1.y], ga1, gx=gin, add=add, mask=1, masked=1, **kw(a1.name)))
            p.names += [ga2, ga1, gin]
            gy, gpre, masked = gin, gin, 1
    p.backward = todo


def _prepare_bn(case, v, code):
    shape, t = tuple(v["x"].shape), torch.bfloat16
    p = Program({n: (shape, t) for n in ("x", "res", "bn", "add", "relu", "gy", "g:add", "g:x")})
    for n in ("x", "res", "gy"):
        p.put(n, v[n])
    p.keep.append(v)
    p.case, p.evict, p.rebuild, p.loss = case, [], None, None
    same = dict(dtype=code, N=case["N"], H=case["H"], W=case["W"], Cin=case["C"], Cout=case["C"], R=1, S=1, stride=1, pad=0, relu=0)
    i = p.ids
    bn = dl.LayerDesc(x=i["x"], res=dl.NO_TENSOR, y=i["bn"], scale=v["gamma"].data_ptr(), shift=v["beta"].data_ptr(), op=dl.OP_BATCHNORM,
                      eps=EPS, **same)
    add = dl.LayerDesc(x=i["bn"], res=i["res"], y=i["add"], op=dl.OP_ADD, **same)
    relu = dl.LayerDesc(x=i["add"], res=dl.NO_TENSOR, y=i["relu"], op=dl.OP_RELU, **same)
    p.forward = dl.layer_array([bn, add, relu])
    # the mask of the backward pass is the stored residual input's sign: an activation that an earlier pass stored
    stored = dl.LayerDesc(x=i["x"], res=dl.NO_TENSOR, y=i["res"], op=dl.OP_RELU, **same)
    p.gw = {"bn": torch.zeros(2 * case["C"], device=DEV)}
    p.backward = [_bwd(p, stored, "gy", gx="g:add"), _bwd(p, bn, "g:add", gx="g:x", gw=p.gw["bn"])]
    p.names = ["bn", "add", "relu", "g:add", "g:x"]
    torch.cuda.synchronize()
    return p


def run(p):
    p.begin()
    d = p.d
    if p.forward is not None:
        d.recompute_segment(p.forward)
        if p.loss is not None:
            d.recompute_segment(p.loss)
    if p.rebuild is not None:
        for t in p.evict:
            d.release(t, dl.EV_EVICT)
        d.recompute_segment(p.rebuild)
    if p.backward is not None:
        d.backward_segment(p.backward)
        d.backward_join()
    res = {n: p.view(n) for n in p.names}
    res.update(("gw:" + n, g) for n, g in p.gw.items())
    return res


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    k = case["kind"]
    if k == "bn":
        n = case["N"] * case["H"] * case["W"] * case["C"] * 2
        return {"bytes": 8 * n, "flops": 0}                    # x, res, gy in; bn, add, relu, g:add, g:x out
    es = 4 if case.get("dtype") == "f32" else 2
    layers = _layers(case)
    params = lambda l: l.Cout * l.R * l.S * l.Cin if l.kind in ("conv", "fc", "linear") else 0    # noqa: E731
    nbytes = flops = 0
    x0 = layers[0].in_elems() * es
    fwd = k != "stem" and case.get("do") != "backward"
    back = k in ("stem", "head") or case.get("do") in ("backward", "both")
    if fwd:
        nbytes += x0 + sum(l.out_elems() * es + params(l) * es for l in layers)
        flops += sum(l.flops for l in layers)
        if case.get("do") == "forward":                        # the internal tensors a second time, from the blocks' inputs
            inner = [l for l in layers if not l.y.endswith(".out")]
            nbytes += sum(l.in_elems() * es for l in inner if l.y.endswith(".a1")) + sum((l.out_elems() + params(l)) * es for l in inner)
            flops += sum(l.flops for l in inner)
    if back and k == "blocks":
        nbytes += x0 * 2 + sum(params(l) * (es + 4) for l in layers)                # x0 in, its gradient out
        for l in layers:
            if l.y.endswith(".sc"):
                continue
            last = l is layers[-1]
            nbytes += l.out_elems() * es * (3 if last else 2)  # stored activation in; gradient out (the last: dL/dy in, masked out)
        flops += 2 * sum(l.flops for l in layers)
    elif k == "stem":
        stem, pool = layers
        nbytes += x0 + stem.out_elems() * 2 * es + pool.out_elems() * es + params(stem) * 4
        flops += stem.flops
    elif k == "head":
        nbytes += layers[0].in_elems() * es + layers[1].in_elems() * es + layers[1].out_elems() * es + params(layers[1]) * 4
        flops += 2 * layers[1].flops
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """About four times the largest distance from `exact` seen on an MI355X: fp32 7.4e-7; a bf16 layer stored once
    1.7e-3 to 2.3e-3; a block's backward 3.9e-3, three blocks' 7.5e-3 (roundings travel); the whole network 9.4e-3."""
    k = case["kind"]
    if case.get("dtype") == "f32":
        return {"rel": 3e-6}
    if k == "resnet" or (k == "blocks" and case["do"] != "forward" and case["blocks"] > 1):
        return {"rel": 3e-2}
    return {"rel": 1.6e-2 if k == "blocks" and case["do"] != "forward" else 1e-2}


# ------------------------------------------------------------------ the same in 64 bits

def _conv(x, w, stride, pad):
    N, H, W, C = x.shape
    K, R, S, _ = w.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    y = torch.zeros(N * P * Q, K, dtype=torch.float64, device=x.device)
    for r in range(R):
        for s in range(S):
            y.addmm_(xp[:, r:r + stride * (P - 1) + 1:stride, s:s + stride * (Q - 1) + 1:stride].reshape(-1, C), w[:, r, s].t())
    return y.view(N, P, Q, K)


def _conv_back(x, w, gy, stride, pad, need_gx=True):
    """(dL/dx, dL/dw) of _conv."""
    N, H, W, C = x.shape
    K, R, S, _ = w.shape
    P, Q = gy.shape[1:3]
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    g2 = gy.reshape(-1, K)
    gw = torch.zeros(K, R, S, C, dtype=torch.float64, device=x.device)
    gp = torch.zeros_like(xp) if need_gx else None
    for r in range(R):
        for s in range(S):
            at = (slice(None), slice(r, r + stride * (P - 1) + 1, stride), slice(s, s + stride * (Q - 1) + 1, stride))
            gw[:, r, s] = g2.t() @ xp[at].reshape(-1, C)
            if need_gx:
                gp[at] += (g2 @ w[:, r, s]).view(N, P, Q, C)
    return (gp[:, pad:pad + H, pad:pad + W] if need_gx else None), gw


def _fold(v, l):
    scale = v["gamma:" + l.name].double() / torch.sqrt(v["var:" + l.name].double() + EPS)
    return scale, v["beta:" + l.name].double() - v["mean:" + l.name].double() * scale


def _forward_layer(l, v, x, res):
    if l.kind == "conv":
        scale, shift = _fold(v, l)
        y = _conv(x, v["w:" + l.name].double(), l.stride, l.pad) * scale + shift
        if res is not None:
            y = y + res
        return y.relu() if l.relu else y
    if l.kind in ("fc", "linear"):
        y = x @ v["w:" + l.name].double().t() + v["bias:" + l.name].double()
        if res is not None:
            y = y + res
        return torch.nn.functional.gelu(y) if l.act == "gelu" else y
    if l.kind == "maxpool":
        return torch.nn.functional.max_pool2d(x.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1)
    if l.kind == "avgpool":
        return x.mean((1, 2), keepdim=True)
    if l.kind == "attention":
        q, kk, vv = (u.reshape(l.N, l.H, l.R, 64).transpose(1, 2).contiguous() for u in x.reshape(l.N, l.H, 3 * l.Cout).split(l.Cout, -1))
        out = torch.empty_like(q)
        for n in range(l.N):
            out[n] = torch.softmax(q[n] @ kk[n].transpose(-1, -2).contiguous() / 8, -1) @ vv[n]
        return out.transpose(1, 2).reshape(l.N, l.H, 1, l.Cout)
    mu = x.mean(-1, keepdim=True)
    var = (x - mu).square().mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(var + synth.LN_EPS) * v["gamma:" + l.name].double() + v["beta:" + l.name].double()


def exact(case, seed):
    """Tensors that the interface stores between layers are read as they are stored (in the case's type)."""
    v = _inputs(case, seed)
    t, k = _tdtype(case), case["kind"]
    stored = lambda y: y.to(t).double()                                            # noqa: E731
    if k == "bn":
        return _exact_bn(v, stored)
    layers = _layers(case)
    res, val = {}, {"x0": v["x0"].double()}
    fwd = k != "stem" and case.get("do") != "backward"
    if fwd:
        for l in layers:
            y = _forward_layer(l, v, val[l.x], val[l.res] if l.res else None)
            val[l.y] = stored(y)
            if k != "resnet" or l.y.endswith(".out") or l.y == "logits":
                res[l.y] = y
            if k == "resnet" and l.y.endswith(".out"):                             # nothing reads what came before
                val = {l.y: val[l.y]}
    if k in ("head", "resnet"):
        z = val["logits"].reshape(case["N"], 1000)
        res["loss"] = torch.nn.functional.cross_entropy(z, v["labels"]).reshape(1)
    if k == "head":
        gz = torch.softmax(z, -1)
        gz[torch.arange(case["N"], device=DEV), v["labels"]] -= 1
        gz /= case["N"]
        res["g:logits"] = gz
        gz = stored(gz)
        a = val["avgpool"].reshape(case["N"], 2048)
        res["g:avgpool"] = gz @ v["w:fc"].double()
        hw = case["H"] * case["W"]
        res["g:x0"] = (stored(res["g:avgpool"]) / hw).view(-1, 1, 1, 2048).expand(-1, case["H"], case["W"], -1)
        res["gw:fc"] = torch.cat([(gz.t() @ a).reshape(-1), gz.sum(0)])
    elif k == "stem":
        x = v["saved:stem"].double()
        N, H, W, C = x.shape
        P, Q = layers[1].P, layers[1].Q
        xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1), value=-math.inf)
        best = torch.full((N, P, Q, C), -math.inf, dtype=torch.float64, device=DEV)
        which = torch.zeros((N, P, Q, C), dtype=torch.uint8, device=DEV)
        win = lambda u, j: u[:, j // 3:j // 3 + 2 * P - 1:2, j % 3:j % 3 + 2 * Q - 1:2]           # noqa: E731
        for j in range(9):                                                         # the first maximum in scan order
            c = win(xp, j)
            which = torch.where(c > best, torch.tensor(j, dtype=torch.uint8, device=DEV), which)
            best = torch.maximum(best, c)
        gp = torch.zeros_like(xp)
        gy = v["gy"].double()
        for j in range(9):
            win(gp, j).add_(gy * (which == j))
        g = gp[:, 1:1 + H, 1:1 + W] * (x > 0)
        res["g:stem"] = g
        scale, _ = _fold(v, layers[0])
        _, gw = _conv_back(val["x0"], v["w:stem"].double(), stored(g), 2, 3, need_gx=False)
        res["gw:stem"] = gw * scale.view(-1, 1, 1, 1)
    elif k == "blocks" and case["do"] != "forward":
        act = lambda n: v["saved:" + n].double() if "saved:" + n in v else v["x0"].double()       # noqa: E731
        by = {l.y: l for l in layers}
        g = v["gy"].double() * (act(layers[-1].y) > 0)

        def back(l, gpre):
            scale, _ = _fold(v, l)
            gx, gw = _conv_back(act(l.x), v["w:" + l.name].double() * scale.view(-1, 1, 1, 1), gpre, l.stride, l.pad)
            res["gw:" + l.name] = gw * scale.view(-1, 1, 1, 1)
            return gx

        for b in range(case["blocks"], 0, -1):
            q = "b%d" % b
            a1, a2, out = by[q + ".a1"], by[q + ".a2"], by[q + ".out"]
            ga2 = back(out, g) * (act(a2.y) > 0)
            add = g
            if q + ".sc" in by:
                add = stored(back(by[q + ".sc"], g))
            ga1 = back(a2, stored(ga2)) * (act(a1.y) > 0)
            gin = (back(a1, stored(ga1)) + add) * (act(a1.x) > 0)
            res["g:" + a2.y], res["g:" + a1.y], res["g:" + a1.x + ":in"] = ga2, ga1, gin
            g = stored(gin)
    return res


def _exact_bn(v, stored):
    x, C = v["x"].double(), v["gamma"].numel()
    mu, var = x.mean((0, 1, 2)), x.var((0, 1, 2), unbiased=False)
    sd = torch.sqrt(var + EPS)
    y = (x - mu) / sd * v["gamma"].double() + v["beta"].double()
    a = stored(y) + v["res"].double()
    g = v["gy"].double() * (v["res"].double() > 0)
    M = x.numel() // C
    sg, sgx = g.sum((0, 1, 2)), (g * (x - mu)).sum((0, 1, 2))
    gx = v["gamma"].double() / sd * (g - sg / M - (x - mu) * sgx / (sd * sd * M))
    return {"bn": y, "add": a, "relu": stored(a).relu(), "g:add": g, "g:x": gx, "gw:bn": torch.cat([sgx / sd, sg])}
