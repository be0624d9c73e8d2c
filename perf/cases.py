"""Performance cases of the elastic selective training step, through the C ABI's Python binding.

A case is one model on one GPU and the call that its user repeats: a masked training step (forward, loss,
weight gradients of the selected tensors, gradient passing down to the input-most of them, optimizer update)
or an evaluation of the tensors' importance (full forward and backward pass, then one reduction over all
weights).  The weights, optimizer state and gradients of a model lie in one arena each, tensors of the same role
(all `qkv.W`, all `ln1.g`, ...) beside each other.
"""
import math
import random

import numpy as np
import torch

from paper_2312_14227_amd import binding as et

RESNET50 = dict(stem=64, blocks=(3, 4, 6, 3), planes=(64, 128, 256, 512))
VGG16 = dict(convs=(2, 2, 3, 3, 3), widths=(64, 128, 256, 512, 512), fc=(4096, 4096))
# (expansion, channels, blocks, stride of the first)
MOBILENETV2 = dict(stem=32, last=1280, settings=((1, 16, 1, 1), (6, 24, 2, 2), (6, 32, 3, 2), (6, 64, 4, 2), (6, 96, 3, 1),
                                                 (6, 160, 3, 2), (6, 320, 1, 1)))
CLASSES = 200   # of the convolutional models and, where a case says nothing else, of the transformers


def _vit(name, batch, tokens, width, blocks, op="train", reach=1.0, pick=1.0, patch_dim=768, classes=CLASSES, mlp=None):
    return dict(name=name, model="vit", op=op, batch=batch, tokens=tokens, patch_dim=patch_dim, width=width, heads=width // 64,
                mlp=mlp or 4 * width, blocks=blocks, classes=classes, reach=reach, pick=pick)


def _conv(name, model, batch, image, op="train", reach=1.0, pick=1.0):
    return dict(name=name, model=model, op=op, batch=batch, image=image, reach=reach, pick=pick)


def listed():
    """`reach`: the part of the tensor chain, counted from the output, that the mask reaches into; `pick`: the share of
    the tensors in that part that it selects.  Selecting for half of the full step's time leaves masks of the kind
    (0.38, 0.4) on a transformer and somewhat deeper ones on the ResNet; 1, 1 is full training."""
    return [
        # The smallest model, float32, batch 32, full training: a step of a dozen tiny launches, all latency.
        dict(name="mlp_b32_full", model="mlp", op="train", batch=32, d_in=256, hidden=256, layers=4, classes=10, reach=1.0, pick=1.0),
        # A small transformer with ragged sizes in every product (3 images, width 192, mlp 320, 56 classes), full training.
        _vit("vit_small_b3_full", 3, 197, 192, 2, patch_dim=200, classes=56, mlp=320),
        # On-device fine-tuning: the base transformer at batch 4, a mask for half the time; also the micro-batch of an
        # importance evaluation.
        _vit("vit_b_b4_half", 4, 197, 768, 12, reach=0.38, pick=0.4),
        # The headline workload: base transformer, batch 64, half of the time.
        _vit("vit_b_b64_half", 64, 197, 768, 12, reach=0.38, pick=0.4),
        # The same with every tensor selected: full training, the denominator of every ratio.
        _vit("vit_b_b64_full", 64, 197, 768, 12),
        # Importance evaluation on the same batch, once per period.
        _vit("vit_b_b64_importance", 64, 197, 768, 12, op="importance"),
        # The large transformer, batch 32, half of the time: the longest chain and the most weights.
        _vit("vit_l_b32_half", 32, 197, 1024, 24, reach=0.38, pick=0.4),
        # Higher-resolution images on a narrow transformer: 577 tokens (24 x 24 patches + CLS), batch 8, full training.
        _vit("vit_577_b8_full", 8, 577, 384, 12),
        # ResNet-50, batch 32, half of the time.
        _conv("resnet50_b32_half", "resnet50", 32, 224, reach=0.6, pick=0.4),
        # ResNet-50 on few images of another size, full training: odd feature maps (50, 25, 13, 7) and ragged row counts.
        _conv("resnet50_b6_i200_full", "resnet50", 6, 200),
        # VGG16, batch 32, fine-tuning its last stage and its linear layers (123 of 135 million weights).
        _conv("vgg16_b32_top", "vgg16", 32, 224, reach=0.37, pick=0.6),
        # MobileNetV2, batch 32, full training: some five hundred short launches.
        _conv("mobilenetv2_b32_full", "mobilenetv2", 32, 224),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the ranges above; batches, image sizes and token counts over their logarithm, whatever they divide."""
    while True:
        mask = dict(reach=1.0, pick=1.0) if rng.random() < 0.35 else dict(reach=rng.uniform(0.1, 0.9), pick=rng.uniform(0.1, 0.9))
        op = "importance" if rng.random() < 0.12 else "train"
        if op == "importance":
            mask = dict(reach=1.0, pick=1.0)
        u = rng.random()
        if u < 0.5:
            width = 64 * rng.choice((3, 4, 6, 8, 10, 12, 16))
            case = _vit("", _log_int(rng, 1, 80), rng.choice((197, _log_int(rng, 17, 640))), width, rng.randint(2, 16), op=op,
                        patch_dim=8 * rng.randint(24, 100), classes=8 * rng.randint(2, 40), mlp=rng.choice((4 * width, 8 * rng.randint(40, 400))),
                        **mask)
        elif u < 0.64:
            case = _conv("", "resnet50", _log_int(rng, 1, 40), rng.choice((224, rng.randint(96, 256))), op=op, **mask)
        elif u < 0.76:
            # masks that end in the last stage: in front of its pooling, near-ties in bf16 let two correct evaluations pick other
            # taps, and their gradients are 5 per cent apart
            case = _conv("", "vgg16", _log_int(rng, 1, 36), 32 * rng.randint(3, 8), reach=rng.uniform(0.1, 0.37), pick=rng.uniform(0.1, 0.9))
        elif u < 0.88:
            case = _conv("", "mobilenetv2", _log_int(rng, 1, 48), rng.choice((224, rng.randint(96, 256))), op=op, **mask)
        else:
            case = dict(model="mlp", op=op, batch=_log_int(rng, 4, 512), d_in=_log_int(rng, 64, 1024), hidden=_log_int(rng, 64, 1024),
                        layers=rng.randint(2, 8), classes=rng.randint(2, 200), **mask)
        case.pop("name", None)
        if work(case)["flops"] <= 4.2e12 and (case["model"] != "mobilenetv2" or case["batch"] * case["image"] ** 2 <= 48 * 224 * 224):
            return case


# ---------------------------------------------------------------------------------------------------- the models
def _chain(case):
    """[(role, shape, kind, rows)] in chain order: kind "matrix" (rows = the rows of the product it takes part in), "vector"
    or "depthwise"; the role names the tensors that lie beside each other."""
    B, out = case["batch"], []
    if case["model"] == "mlp":
        dims = [case["d_in"]] + [case["hidden"]] * (case["layers"] - 1) + [case["classes"]]
        return [("fc.W" if i + 1 < case["layers"] else "head.W", (dims[i + 1], dims[i]), "matrix", B) for i in range(case["layers"])]
    if case["model"] == "vit":
        T, D, F, P, C = (case[k] for k in ("tokens", "width", "mlp", "patch_dim", "classes"))
        out = [("patch.W", (D, P), "matrix", B * (T - 1)), ("patch.b", (D,), "vector", 0), ("cls", (D,), "vector", 0), ("pos", (T, D), "vector", 0)]
        for l in range(case["blocks"]):
            # behind the last block only the CLS row is read: its queries, projection and MLP exist for B rows
            M = B * T
            m = B if l + 1 == case["blocks"] else M
            out += [("ln1.g", (D,), "vector", 0), ("ln1.b", (D,), "vector", 0),
                    ("qkv.W", (3 * D, D), "matrix", (2 * M + m) / 3), ("qkv.b", (3 * D,), "vector", 0),
                    ("proj.W", (D, D), "matrix", m), ("proj.b", (D,), "vector", 0),
                    ("ln2.g", (D,), "vector", 0), ("ln2.b", (D,), "vector", 0),
                    ("fc1.W", (F, D), "matrix", m), ("fc1.b", (F,), "vector", 0), ("fc2.W", (D, F), "matrix", m), ("fc2.b", (D,), "vector", 0)]
        return out + [("lnf.g", (D,), "vector", 0), ("lnf.b", (D,), "vector", 0), ("head.W", (C, D), "matrix", B), ("head.b", (C,), "vector", 0)]
    side = case["image"]
    if case["model"] == "resnet50":
        a = RESNET50
        side = (side - 1) // 2 + 1
        cin = a["stem"]
        out = [("stem.W", (cin, 7, 7, 3), "matrix", B * side * side), ("stem.g", (cin,), "vector", 0), ("stem.b", (cin,), "vector", 0)]
        side = (side - 1) // 2 + 1
        for s, (n, p) in enumerate(zip(a["blocks"], a["planes"])):
            for k in range(n):
                full = B * side * side
                if k == 0 and s > 0:
                    side = (side - 1) // 2 + 1
                M = B * side * side
                for name, shape, rows in (("c1", (p, 1, 1, cin), full), ("c2", (p, 3, 3, p), M), ("c3", (4 * p, 1, 1, p), M)) + (
                        (("sc", (4 * p, 1, 1, cin), M),) if k == 0 else ()):
                    out += [(name + ".W", shape, "matrix", rows), (name + ".g", shape[:1], "vector", 0), (name + ".b", shape[:1], "vector", 0)]
                cin = 4 * p
        return out + [("head.W", (CLASSES, cin), "matrix", B), ("head.b", (CLASSES,), "vector", 0)]
    if case["model"] == "vgg16":
        cin = 3
        for s, (w, n) in enumerate(zip(VGG16["widths"], VGG16["convs"])):
            for k in range(n):
                name = "first" if cin == 3 else "pool%d" % s if k + 1 == n else "s%d" % s   # pool: the one in front of the stage's pooling
                out += [(name + ".W", (w, 3, 3, cin), "matrix", B * side * side), (name + ".b", (w,), "vector", 0)]
                cin = w
            side //= 2
        fin = side * side * cin
        for j, f in enumerate(VGG16["fc"] + (CLASSES,)):
            out += [("fc%d.W" % j, (f, fin), "matrix", B), ("fc%d.b" % j, (f,), "vector", 0)]
            fin = f
        return out
    a = MOBILENETV2
    side = (side - 1) // 2 + 1
    cin = a["stem"]

    def unit(name, shape, kind, rows):
        return [(name + ".W", shape, kind, rows), (name + ".g", shape[:1], "vector", 0), (name + ".b", shape[:1], "vector", 0)]

    out = unit("stem", (cin, 3, 3, 3), "matrix", B * side * side)
    for (t, c, n, s) in a["settings"]:
        for k in range(n):
            hid = t * cin
            if t != 1:
                out += unit("exp", (hid, 1, 1, cin), "matrix", B * side * side)
            if k == 0:
                side = (side - 1) // s + 1
            out += unit("dw", (hid, 3, 3, 1), "depthwise", B * side * side)
            # a projection whose output joins a shortcut, and one that opens a stage
            out += unit("join" if k else "proj", (c, 1, 1, hid), "matrix", B * side * side)
            cin = c
    out += unit("last", (a["last"], 1, 1, cin), "matrix", B * side * side)
    return out + [("head.W", (CLASSES, a["last"]), "matrix", B), ("head.b", (CLASSES,), "vector", 0)]


def _mask(case, n):
    first = n - max(1, int(round(case["reach"] * n)))
    rng = random.Random(n)
    m = [i >= first and (case["pick"] >= 1.0 or rng.random() < case["pick"]) for i in range(n)]
    m[first] = True
    return m


def _desc(case):
    b = case["batch"]
    if case["model"] == "mlp":
        return et.make_desc(et.ET_MLP, et.ET_F32, b, dims=(case["d_in"],) + (case["hidden"],) * (case["layers"] - 1) + (case["classes"],))
    if case["model"] == "vit":
        return et.make_desc(et.ET_VIT, et.ET_BF16, b, tokens=case["tokens"], patch_dim=case["patch_dim"], width=case["width"], heads=case["heads"],
                            mlp=case["mlp"], blocks=case["blocks"], classes=case["classes"])
    common = dict(classes=CLASSES, image=case["image"], in_ch=3)
    if case["model"] == "resnet50":
        return et.make_desc(et.ET_RESNET, et.ET_BF16, b, stem=RESNET50["stem"], stage_blocks=RESNET50["blocks"], planes=RESNET50["planes"], **common)
    if case["model"] == "vgg16":
        return et.make_desc(et.ET_VGG, et.ET_BF16, b, dims=VGG16["fc"] + (CLASSES,), stage_blocks=VGG16["convs"], planes=VGG16["widths"], **common)
    s = MOBILENETV2["settings"]
    return et.make_desc(et.ET_MOBILENET, et.ET_BF16, b, stem=MOBILENETV2["stem"], last=MOBILENETV2["last"], stage_blocks=[n for (_, _, n, _) in s],
                        planes=[c for (_, c, _, _) in s], expand=[t for (t, _, _, _) in s], strides=[st for (_, _, _, st) in s], **common)


def _initial(case, role, shape, gen):
    """Initial values.  Transformers and perceptrons are drawn as the workloads draw them (truncated normals of 0.02; He-normal).

    In the convolutional models three channels of four are mostly on and every fourth is mostly off: shifts of about three standard
    deviations, weights that cancel the mean of their inputs.  Channels balanced on the edge of their ReLU, which is what zero
    shifts give, make two correct bf16 evaluations of a deep stack disagree by several per cent in the gradients (each
    stored value rounds differently, and a fraction of the masks follows), so that no results could be compared.
    In front of a max pooling, where only the largest of four values passes a gradient, the shift is smaller: the finer bf16 grid
    leaves fewer near-ties for the choice."""
    leaf = role.split(".")[-1]
    normal = lambda std: torch.randn(shape, generator=gen, device="cuda") * std  # noqa: E731
    if case["model"] == "vit":
        if leaf == "g":
            return 1.0 + normal(0.1)
        return normal(0.02) if leaf == "b" else normal(1.0).clamp_(-2.0, 2.0) * 0.02
    if case["model"] == "mlp":
        return normal(math.sqrt(2.0 / shape[1]))
    on = lambda n: torch.arange(n, device="cuda") % 4 != 0  # noqa: E731
    if leaf == "g":
        # the residual branches join their stream at a quarter
        return {"c3.g": 0.25, "join.g": 0.25, "stem.g": 0.7}.get(role, 1.0) * (1.0 + normal(0.02))
    if leaf == "b":
        mean_on, mean_off = {"c3.b": (0.0, -1.0), "join.b": (0.0, 0.0), "proj.b": (0.0, 0.0), "head.b": (0.0, 0.0), "fc%d.b" % len(VGG16["fc"]): (0.0, 0.0)}.get(
            role, (0.7, -3.0) if role.startswith("pool") else (2.2, -2.2) if case["model"] == "vgg16" and not role.startswith("fc") else (3.0, -3.0))
        return torch.where(on(shape[0]), mean_on, mean_off) + normal(0.02)
    if role == "dw.W":
        w = normal(0.2)
        w[:, 1, 1] += 0.6
        return w - w.mean(dim=(1, 2), keepdim=True)
    fan = math.prod(shape[1:])
    linear_input = role in ("first.W", "exp.W", "last.W") or shape[-1] == 3
    if linear_input:
        return normal(math.sqrt(0.5 / fan))
    w = normal(math.sqrt((1.7 if case["model"] == "vgg16" else 2.0 if role in ("join.W", "proj.W") else 1.4) / fan))
    return w - (w * on(shape[-1])).sum(dim=-1, keepdim=True) / on(shape[-1]).sum()


class _Model:
    """What a training program holds: the context, the arenas of weights, optimizer state and gradients, the workspace."""

    def __init__(self, case, seed):
        self.ctx = None
        gen = torch.Generator(device="cuda").manual_seed(seed)
        chain = _chain(case)
        self.dtype = torch.float32 if case["model"] == "mlp" else torch.bfloat16
        offset, total, self.roles = [0] * len(chain), 0, {}
        for role in dict.fromkeys(r for r, *_ in chain):
            begin = total
            for i, (r, shape, _, _) in enumerate(chain):
                if r == role:
                    offset[i] = total
                    total += (math.prod(shape) + 63) // 64 * 64
            self.roles[role] = slice(begin, total)
        self.mask = np.array(_mask(case, len(chain)), dtype=np.uint8)
        self.w = torch.zeros(total, dtype=self.dtype, device="cuda")
        self.grad = torch.zeros(total, device="cuda")
        for (role, shape, _, _), o in zip(chain, offset):
            self.w[o:o + math.prod(shape)] = _initial(case, role, shape, gen).reshape(-1).to(self.dtype)
        self.ctx = et.et_create(_desc(case), torch.cuda.current_stream().cuda_stream)
        assert [et.et_tensor_info(self.ctx, i)[0] for i in range(et.et_num_tensors(self.ctx))] == [math.prod(s) for _, s, _, _ in chain]
        slots = et.et_state_slots(self.ctx)
        self.state = [self.w.float() if s == 0 and slots == 3 else torch.zeros(total, device="cuda") for s in range(slots)]
        need = et.et_workspace_bytes(self.ctx)
        self.ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
        at = lambda t: [t.data_ptr() + t.element_size() * o for o in offset]  # noqa: E731
        per_slot = [at(s) for s in self.state]
        et.et_bind(self.ctx, at(self.w), [p[i] for i in range(len(chain)) for p in per_slot], at(self.grad), -(-self.ws.data_ptr() // 256) * 256, need)
        B = case["batch"]
        self.x = torch.randn({"mlp": (B, case.get("d_in")), "vit": (B, case.get("tokens", 2) - 1, case.get("patch_dim"))}.get(
            case["model"], (B, case.get("image"), case.get("image"), 3)), generator=gen, device="cuda").to(self.dtype)
        self.y = torch.randint(0, case.get("classes", CLASSES), (B,), generator=gen, device="cuda", dtype=torch.int32)
        self.opt = et.et_opt()
        self.opt.kind = et.ET_ADAM if case["model"] == "vit" else et.ET_SGDW
        # fine-tuning rates between 1e-5 and 1e-4 (a plain stack of convolutions oscillates from step to step at 1e-4)
        self.opt.lr, self.opt.beta1, self.opt.beta2, self.opt.eps = 1e-4 if case["model"] == "vit" else 1e-5, 0.9, 0.999, 1e-8
        self.opt.momentum, self.opt.wd, self.opt.step = 0.9, 5e-4, 0
        if case["op"] == "importance":
            self.snapshot = (self.w.float() + 1e-3 * torch.randn(total, generator=gen, device="cuda")).to(self.dtype)
            self.snapshot_ptrs = at(self.snapshot)

    def by_role(self, arena):
        return {role: arena[part] for role, part in self.roles.items()}

    def __del__(self):
        if self.ctx is not None and torch is not None:
            torch.cuda.synchronize()
            et.et_destroy(self.ctx)


def prepare(case, seed):
    return {"op": case["op"], "model": _Model(case, seed)}


def run(state):
    s = state["model"]
    if state["op"] == "importance":
        values = et.et_importance(s.ctx, s.x.data_ptr(), s.y.data_ptr(), s.snapshot_ptrs)
        return {"importance": values, "grad": s.by_role(s.grad)}
    s.opt.step += 1
    et.et_train_step(s.ctx, s.x.data_ptr(), s.y.data_ptr(), s.mask, s.opt, want_loss=False)
    moments = s.state[-2:] if s.opt.kind == et.ET_ADAM else s.state[-2:-1]
    out = {"grad": s.by_role(s.grad), "w": s.w, "moments": [s.by_role(t) for t in moments]}
    if len(s.state) == 3:
        out["master"] = s.state[0]
    return out


# ---------------------------------------------------------------------------------------------------- work and tolerance
def work(case):
    chain = _chain(case)
    n = len(chain)
    train = case["op"] == "train"
    mask = _mask(case, n) if train else [True] * n
    first = mask.index(True)
    size = [math.prod(s) for _, s, _, _ in chain]
    flops = 0.0
    for i, (_, shape, kind, rows) in enumerate(chain):
        one = 2.0 * rows * (9 * shape[0] if kind == "depthwise" else size[i] if kind == "matrix" else 0)
        flops += one * (1 + mask[i] + (i > first))
    if case["model"] == "vit":
        B, T, D = case["batch"], case["tokens"], case["width"]
        for l in range(case["blocks"]):
            queries = 1 if l + 1 == case["blocks"] else T
            flops += 4.0 * B * queries * T * D * (3 if first < 4 + 12 * l + 4 else 1)
    wb = 4 if case["model"] == "mlp" else 2
    x = case["batch"] * (case["d_in"] * 4 if case["model"] == "mlp" else 2 * (case["tokens"] - 1) * case["patch_dim"] if case["model"] == "vit"
                         else 2 * 3 * case["image"] ** 2)
    picked = sum(v for v, m in zip(size, mask) if m)
    moments = 2 if case["model"] == "vit" else 1
    per_picked = 4 + ((2 * 4 * moments + (4 if wb == 4 else 2 * 4 + 2)) if train else wb)
    return {"bytes": x + wb * sum(size) + per_picked * picked, "flops": flops}


def tolerance(case):
    """Measured by evaluating every listed case and some drawn ones twice, the second time with the features of the first product in
    another order (the inputs of a perceptron or a transformer, the image channels, the stem's output channels), results put back
    in place: float32 sums 7e-7 at most (largest single difference 1e-5 of the root mean square); bf16 gradients and moments
    0.005 to 0.013 on the transformers (0.6 at most for a single value), 0.008 to 0.012 on ResNet-50, 0.003 to 0.019 on VGG16 (the latter over six steps),
    0.01 on MobileNetV2; importances 0.01."""
    if case["model"] == "mlp":
        return {"rel": 3e-6, "max": 1e-4}
    return {"rel": 0.03, "max": 0.9}
