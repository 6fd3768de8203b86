"""Performance cases: the programs a user of this library runs, from one small layer to whole networks.

Every case is a typed graph declared, planned and prepacked once (what a program keeps) and then run through `Plan.run` or
`Plan.run_recurrent` on device tensors, the way `paper_1810_00952_amd.harness.Session` does.  Sizes are those of the repository's
workloads, tests and benchmark, or ragged neighbours of them; `draw` spreads over the same families."""
import math

import torch

from paper_1810_00952_amd import Context, Graph, Plan

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
DEVICE = "cuda:0"


# ---- the cases ---------------------------------------------------------------------------------------------------------
def listed():
    return [
        # a two-layer classifier on MNIST-shaped rows: the smallest call, where launches and latency are the time
        dict(name="mlp_f32_b32", family="mlp", dtype="f32", batch=32, d_in=784, d_hidden=128, d_out=10),
        # one convolution layer of a single image, f32: interactive inference
        dict(name="conv_f32_b1", family="conv", dtype="f32", batch=1, cin=64, cout=64, h=56, w=56, k=3, stride=1, pad=1, residual=False),
        # the small convolutional network of the paper's example, a batch of 64 through the whole model (logits)
        dict(name="lenet_f32_b64", family="lenet", dtype="f32", batch=64),
        # a convolution layer whose channel counts and rows are no multiples of any tile, with a skip connection
        dict(name="conv_bf16_ragged", family="conv", dtype="bf16", batch=17, cin=96, cout=136, h=29, w=29, k=3, stride=1, pad=1, residual=True),
        # a classifier-sized dense layer whose sizes are no multiples of a tile
        dict(name="dense_bf16_ragged", family="dense", dtype="bf16", m=1000, n=1000, k=784),
        # a dense layer at matrix-multiplication scale
        dict(name="dense_bf16_4096", family="dense", dtype="bf16", m=4096, n=4096, k=4096),
        # the backward pass of a dense layer: both gradients, that of the weights in f32 for the optimizer
        dict(name="dense_grad_bf16", family="dense_grad", dtype="bf16", m=512, n=1000, k=784),
        # the backward pass of a convolution layer, mixed precision, a full batch
        dict(name="conv_grad_bf16_b64", family="conv_grad", dtype="bf16", batch=64, cin=128, cout=128, h=28, w=28, k=3, stride=1, pad=1),
        # the same in f32 on a smaller layer and batch
        dict(name="conv_grad_f32_b32", family="conv_grad", dtype="f32", batch=32, cin=64, cout=64, h=28, w=28, k=3, stride=1, pad=1),
        # bias + skip + ReLU on large activations: memory bandwidth
        dict(name="eltwise_bf16_large", family="eltwise", dtype="bf16", shape0=256, shape1=64, shape2=112, shape3=112),
        # a sequence batch through a recurrent cell: 128 dependent steps
        dict(name="lstm_bf16_b64", family="lstm", dtype="bf16", batch=64, d_in=1024, hidden=1024, steps=128),
        # image classification at serving batch size, the whole network (logits): the headline
        dict(name="resnet18_bf16_b64", family="resnet18", dtype="bf16", batch=64),
    ]


def _log_int(rng, lo, hi, multiple=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, max(1, round(v / multiple)) * multiple))


def draw(rng):
    """One more case of the listed families.  Half of the channel and feature counts are multiples of 8 or 64, as layers are
    usually laid out; the rest are whatever comes."""
    def count(lo, hi):
        m = rng.choice([1, 1, 8, 64])
        return _log_int(rng, max(lo, m), hi, m)

    family = rng.choice(["mlp", "conv", "conv", "lenet", "dense", "dense", "dense_grad", "conv_grad", "conv_grad", "eltwise", "lstm", "resnet18"])
    dtype = rng.choice(["f32", "bf16"])
    if family == "mlp":
        return dict(family=family, dtype=dtype, batch=_log_int(rng, 1, 256), d_in=count(32, 2048), d_hidden=count(16, 1024), d_out=_log_int(rng, 2, 100))
    if family == "lenet":
        return dict(family=family, dtype=dtype, batch=_log_int(rng, 1, 256))
    if family == "resnet18":
        return dict(family=family, dtype=dtype, batch=_log_int(rng, 1, 64 if dtype == "bf16" else 8))
    if family == "dense":
        top = 4096 if dtype == "bf16" else 2048
        return dict(family=family, dtype=dtype, m=_log_int(rng, 8, top), n=count(10, top), k=count(64, top))
    if family == "dense_grad":
        return dict(family=family, dtype=dtype, m=_log_int(rng, 8, 4096), n=count(10, 2048), k=count(16, 2048))
    if family == "eltwise":
        return dict(family=family, dtype=dtype, shape0=_log_int(rng, 1, 128), shape1=count(3, 128), shape2=_log_int(rng, 1, 112), shape3=_log_int(rng, 1, 112))
    if family == "lstm":
        return dict(family=family, dtype=dtype, batch=_log_int(rng, 1, 96), d_in=_log_int(rng, 32, 1024, 16), hidden=_log_int(rng, 32, 1024, 16),
                    steps=_log_int(rng, 4, 96))
    # a layer and its backward pass: up to about 15 GFLOP in bf16, a quarter of that in f32 and in the backward passes
    top = 1.5e10 if family == "conv" and dtype == "bf16" else 4e9
    while True:
        k = rng.choice([1, 3, 3, 3, 5])
        stride = rng.choice([1, 1, 2])
        c = dict(family=family, dtype=dtype, batch=rng.choice([64, 32, _log_int(rng, 1, 64), _log_int(rng, 1, 64)]), cin=count(3 if family == "conv" else 8, 512),
                 cout=count(8, 512), h=rng.randint(7, 57), w=0, k=k, stride=stride, pad=rng.choice([k // 2, k // 2, 0]))
        c["w"] = rng.choice([c["h"], c["h"], rng.randint(7, 57)])
        if family == "conv":
            c["residual"] = rng.random() < 0.5
        if work(c)["flops"] <= top:
            return c


# ---- what a case cannot do without -----------------------------------------------------------------------------------------
def _out(h, k, s, p):
    return (h + 2 * p - k) // s + 1


# the residual network: (name, cin, cout, kernel, stride, pad, input size, what its skip is) of every convolution
def _resnet_layers():
    layers = [("conv1", 3, 64, 7, 2, 3, 224, None)]
    h, cin = 56, 64
    for stage in range(4):
        cout = 64 << stage
        for blk in range(2):
            s = 2 if stage and not blk else 1
            name = f"l{stage + 1}.b{blk}"
            layers.append((name + ".c1", cin, cout, 3, s, 1, h, None))
            if s != 1:
                layers.append((name + ".ds", cin, cout, 1, s, 0, h, None))
            h = _out(h, 3, s, 1)
            layers.append((name + ".c2", cout, cout, 3, 1, 1, h, "skip"))
            cin = cout
    return layers


def work(case):
    f, b = case["family"], {"f32": 4, "bf16": 2}[case["dtype"]]
    if f == "mlp":
        m, i, h, o = case["batch"], case["d_in"], case["d_hidden"], case["d_out"]
        return dict(bytes=b * (m * i + i * h + h * o + m * o) + 4 * (h + o), flops=2 * m * (i * h + h * o))
    if f == "dense":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=b * (m * k + n * k + m * n) + 4 * n, flops=2 * m * n * k)
    if f == "dense_grad":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(bytes=b * (m * n + n * k + m * k + m * k) + 4 * n * k, flops=4 * m * n * k)
    if f in ("conv", "conv_grad"):
        n, c, o, k = case["batch"], case["cin"], case["cout"], case["k"]
        oh, ow = _out(case["h"], k, case["stride"], case["pad"]), _out(case["w"], k, case["stride"], case["pad"])
        x, y, w = n * c * case["h"] * case["w"], n * o * oh * ow, o * c * k * k
        fl = 2 * y * c * k * k
        if f == "conv":
            return dict(bytes=b * (x + w + y * (2 if case["residual"] else 1)) + 4 * o, flops=fl)
        return dict(bytes=b * (y + w + x + x) + 4 * w, flops=2 * fl)
    if f == "lenet":
        n = case["batch"]
        w = 20 * 25 + 50 * 20 * 25 + 800 * 500 + 500 * 10
        return dict(bytes=b * (n * 794 + w) + 4 * 580, flops=2 * n * (20 * 25 * 576 + 50 * 500 * 64 + 800 * 500 + 5000))
    if f == "resnet18":
        n, fl, w = case["batch"], 0, 512 * 1000
        for _, ci, co, k, s, p, h, _ in _resnet_layers():
            fl += 2 * n * _out(h, k, s, p) ** 2 * co * ci * k * k
            w += ci * co * k * k
        return dict(bytes=b * (n * (3 * 224 * 224 + 1000) + w) + 4 * (4800 + 1000), flops=fl + 2 * n * 512 * 1000)
    if f == "eltwise":
        e = case["shape0"] * case["shape1"] * case["shape2"] * case["shape3"]
        return dict(bytes=3 * b * e + 4 * case["shape1"], flops=3 * e)
    m, i, h, t = case["batch"], case["d_in"], case["hidden"], case["steps"]
    return dict(bytes=b * (t * m * (i + h) + 4 * h * (i + h)) + 4 * (4 * h + m * h), flops=t * m * (8 * h * (i + h) + 30 * h))


# ---- inputs: from the seed alone, the values the layers meet in use ----------------------------------------------------------
def _data(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    f, dt = case["family"], TORCH[case["dtype"]]

    def normal(*shape, std=1.0, dtype=dt):
        return (torch.randn(*shape, generator=g, device=DEVICE, dtype=torch.float32) * std).to(dtype)

    def uniform(*shape, bound=0.1, dtype=torch.float32):
        return ((torch.rand(*shape, generator=g, device=DEVICE, dtype=torch.float32) * 2 - 1) * bound).to(dtype)

    if f == "mlp":
        i, h, o = case["d_in"], case["d_hidden"], case["d_out"]
        return dict(x=normal(case["batch"], i), w1=uniform(h, i, bound=(6 / i) ** 0.5, dtype=dt), b1=uniform(h),
                    w2=uniform(o, h, bound=(6 / h) ** 0.5, dtype=dt), b2=uniform(o))
    if f == "dense":
        return dict(x=normal(case["m"], case["k"]), w=uniform(case["n"], case["k"], bound=(6 / case["k"]) ** 0.5, dtype=dt), b=uniform(case["n"]))
    if f == "dense_grad":
        m, n, k = case["m"], case["n"], case["k"]
        return dict(dy=normal(m, n), x=normal(m, k), w=uniform(n, k, bound=(6 / k) ** 0.5, dtype=dt))
    if f in ("conv", "conv_grad"):
        n, ci, co, k = case["batch"], case["cin"], case["cout"], case["k"]
        oh, ow = _out(case["h"], k, case["stride"], case["pad"]), _out(case["w"], k, case["stride"], case["pad"])
        d = dict(x=normal(n, ci, case["h"], case["w"]), w=normal(co, ci, k, k, std=(2 / (ci * k * k)) ** 0.5))
        if f == "conv_grad":
            d["dy"] = normal(n, co, oh, ow)
        else:
            d["b"] = uniform(co)
            if case["residual"]:
                d["r"] = normal(n, co, oh, ow)
        return d
    if f == "lenet":
        d = dict(x=normal(case["batch"], 1, 28, 28))
        for name, shape in (("conv1", (20, 1, 5, 5)), ("conv2", (50, 20, 5, 5)), ("fc1", (500, 800)), ("fc2", (10, 500))):
            fan = math.prod(shape[1:])
            d[name + ".w"], d[name + ".b"] = uniform(*shape, bound=(6 / fan) ** 0.5, dtype=dt), uniform(shape[0])
        return d
    if f == "resnet18":                                 # batch-norm already folded into the weights, as for inference
        d = dict(x=normal(case["batch"], 3, 224, 224))
        for name, ci, co, k, _, _, _, _ in _resnet_layers():
            scale = 1 + uniform(co, 1, 1, 1, bound=0.5)
            d[name + ".w"] = (normal(co, ci, k, k, std=(2 / (ci * k * k)) ** 0.5, dtype=torch.float32) * scale).to(dt)
            d[name + ".b"] = uniform(co)
        d["fc.w"], d["fc.b"] = uniform(1000, 512, bound=(6 / 512) ** 0.5, dtype=dt), uniform(1000)
        return d
    if f == "eltwise":
        s = [case[f"shape{i}"] for i in range(4)]
        return dict(x=normal(*s), r=normal(*s), b=uniform(s[1]))
    i, h, bound = case["d_in"], case["hidden"], case["hidden"] ** -0.5
    return dict(x=normal(case["steps"], case["batch"], i), w=uniform(4 * h, i + h, bound=bound, dtype=dt), b=uniform(4 * h, bound=bound))


# ---- the programs ----------------------------------------------------------------------------------------------------------
class Program:
    """A graph under construction: values by name, one fusion group per `group` call, and what they are bound to."""

    def __init__(self, data):
        self.graph, self.data, self.bound, self.shapes = Graph(Context()), data, {}, {}

    def _new(self, make, name):
        t = self.data[name]
        vid = make("bf16" if t.dtype == torch.bfloat16 else "f32", tuple(t.shape))
        self.bound[vid] = t
        return vid

    def input(self, name):
        return self._new(self.graph.input, name)

    def param(self, name):
        vid = self._new(self.graph.param, name)
        self.shapes[vid] = "param"
        return vid

    def group(self, first, out_type, *then):
        """One fused group: (kind, operands, attrs) for its first call, (kind, more operands, attrs) for those that follow."""
        kind, ins, attrs = first
        op, (v,) = self.graph.op(kind, ins, [out_type], **attrs)
        ops = [op]
        for kind, more, attrs in then:
            op, (v,) = self.graph.op(kind, [v] + more, [out_type], **attrs)
            ops.append(op)
        self.graph.group(ops)
        return v

    def finish(self, *outputs):
        """Plan, prepack the params, allocate outputs [(value, (dtype, shape))] and workspace."""
        for v, _ in outputs:
            self.graph.output(v)
        plan = Plan(self.graph)
        stream = torch.cuda.current_stream().cuda_stream
        for vid, t in self.bound.items():
            if vid in self.shapes and plan.packed_bytes(vid):
                packed = torch.empty(plan.packed_bytes(vid), dtype=torch.uint8, device=DEVICE)
                plan.prepack(vid, t.data_ptr(), packed.data_ptr(), stream)
                self.bound[vid] = packed
        outs = []
        for v, (dtype, shape) in outputs:
            self.bound[v] = torch.empty(shape, dtype=TORCH[dtype], device=DEVICE)
            outs.append(self.bound[v])
        ws = torch.empty(max(256, plan.workspace_bytes()), dtype=torch.uint8, device=DEVICE)
        # "keep": the caller's own tensors stay alive with the state (a packed param replaced its binding)
        return dict(plan=plan, bindings={vid: t.data_ptr() for vid, t in self.bound.items()}, workspace=ws, outputs=outs, keep=(self.bound, self.data))


def prepare(case, seed):
    f, dt, d = case["family"], case["dtype"], _data(case, seed)
    if f == "lstm":
        return _prepare_lstm(case, d)
    p = Program(d)
    bias = lambda name: ("bias_add", [p.param(name)], dict(axis=1))
    relu, tanh = ("relu", [], {}), ("tanh", [], {})
    if f == "mlp":
        th, to = (dt, (case["batch"], case["d_hidden"])), (dt, (case["batch"], case["d_out"]))
        h = p.group(("dense", [p.input("x"), p.param("w1")], {}), th, bias("b1"), relu)
        return p.finish((p.group(("dense", [h, p.param("w2")], {}), to, bias("b2")), to))
    if f == "dense":
        t = (dt, (case["m"], case["n"]))
        return p.finish((p.group(("dense", [p.input("x"), p.param("w")], {}), t, bias("b"), relu), t))
    if f == "dense_grad":
        m, n, k = case["m"], case["n"], case["k"]
        dy, tx, tw = p.input("dy"), (dt, (m, k)), ("f32", (n, k))
        dx = p.group(("dense_grad_x", [dy, p.param("w")], {}), tx)
        dw = p.group(("dense_grad_w", [dy, p.input("x")], dict(out_dtype="f32")), tw)
        return p.finish((dx, tx), (dw, tw))
    if f in ("conv", "conv_grad"):
        k, s = case["k"], (case["stride"],) * 2
        at = dict(stride=s, pad=(case["pad"],) * 2)
        if f == "conv_grad":
            dy, tx, tw = p.input("dy"), (dt, tuple(d["x"].shape)), ("f32", tuple(d["w"].shape))
            dx = p.group(("conv2d_grad_x", [dy, p.param("w")], at), tx)
            dw = p.group(("conv2d_grad_w", [dy, p.input("x")], dict(at, out_dtype="f32")), tw)
            return p.finish((dx, tx), (dw, tw))
        t = (dt, (case["batch"], case["cout"], _out(case["h"], k, s[0], case["pad"]), _out(case["w"], k, s[0], case["pad"])))
        steps = [bias("b")] + ([("add", [p.input("r")], {})] if case["residual"] else []) + [relu]
        return p.finish((p.group(("conv2d", [p.input("x"), p.param("w")], at), t, *steps), t))
    if f == "eltwise":
        t = (dt, tuple(d["x"].shape))
        return p.finish((p.group(("bias_add", [p.input("x"), p.param("b")], dict(axis=1)), t, ("add", [p.input("r")], {}), relu), t))
    if f == "lenet":
        n, y, h = case["batch"], p.input("x"), 28
        for name, c in (("conv1", 20), ("conv2", 50)):
            y = p.group(("conv2d", [y, p.param(name + ".w")], {}), (dt, (n, c, h - 4, h - 4)), bias(name + ".b"), tanh)
            h = (h - 4) // 2
            y = p.group(("maxpool2d", [y], dict(kernel=(2, 2), stride=(2, 2))), (dt, (n, c, h, h)))
        y = p.group(("flatten", [y], {}), (dt, (n, 800)))
        y = p.group(("dense", [y, p.param("fc1.w")], {}), (dt, (n, 500)), bias("fc1.b"), tanh)
        return p.finish((p.group(("dense", [y, p.param("fc2.w")], {}), (dt, (n, 10)), bias("fc2.b")), (dt, (n, 10))))
    n, y, y1, skip = case["batch"], p.input("x"), None, None
    for name, _, co, k, s, pad, h, res in _resnet_layers():
        if name.endswith(".c1"):
            skip = y
        src = skip if name.endswith(".ds") else y1 if res else y
        t = (dt, (n, co, _out(h, k, s, pad), _out(h, k, s, pad)))
        steps = [bias(name + ".b")] + ([("add", [skip], {})] if res else []) + ([] if name.endswith(".ds") else [relu])
        v = p.group(("conv2d", [src, p.param(name + ".w")], dict(stride=(s, s), pad=(pad, pad))), t, *steps)
        if name == "conv1":
            y = p.group(("maxpool2d", [v], dict(kernel=(3, 3), stride=(2, 2), pad=(1, 1))), (dt, (n, 64, 56, 56)))
        elif name.endswith(".ds"):
            skip = v
        elif res:
            y = v
        else:
            y1 = v
    y = p.group(("global_avgpool", [y], {}), (dt, (n, 512, 1, 1)))
    y = p.group(("flatten", [y], {}), (dt, (n, 512)))
    return p.finish((p.group(("dense", [y, p.param("fc.w")], {}), (dt, (n, 1000)), bias("fc.b")), (dt, (n, 1000))))


def _prepare_lstm(case, d):
    dt, m, i, h, t = case["dtype"], case["batch"], case["d_in"], case["hidden"], case["steps"]
    g = Graph(Context())
    x, hin, c, w, b = g.input(dt, (m, i)), g.input(dt, (m, h)), g.input("f32", (m, h)), g.param(dt, (4 * h, i + h)), g.param("f32", (4 * h,))
    o0, (xh,) = g.op("concat", [x, hin], [(dt, (m, i + h))], axis=1)
    o1, (z,) = g.op("dense", [xh, w], [("f32", (m, 4 * h))], out_dtype="f32")
    o2, (z,) = g.op("bias_add", [z, b], [("f32", (m, 4 * h))], axis=1)
    o3, (c2, h2) = g.op("lstm_gates", [z, c], [("f32", (m, h)), (dt, (m, h))])
    g.group([o0, o1, o2, o3])
    g.output(c2)
    g.output(h2)
    plan = Plan(g)
    packed = torch.empty(max(256, plan.packed_bytes(w)), dtype=torch.uint8, device=DEVICE)
    if plan.packed_bytes(w):
        plan.prepack(w, d["w"].data_ptr(), packed.data_ptr(), torch.cuda.current_stream().cuda_stream)
    else:
        packed = d["w"]
    ws = torch.empty(max(256, plan.recurrent_workspace_bytes(t)), dtype=torch.uint8, device=DEVICE)
    return dict(plan=plan, steps=t, roles=dict(x=x, h_in=hin, c_in=c, h_out=h2, c_out=c2), x=d["x"], x_step=m * i * d["x"].element_size(),
                h0=torch.zeros(m, h, dtype=TORCH[dt], device=DEVICE), c=torch.zeros(m, h, dtype=torch.float32, device=DEVICE),
                hs=torch.empty(t, m, h, dtype=TORCH[dt], device=DEVICE), params={w: packed.data_ptr(), b: d["b"].data_ptr()}, workspace=ws, keep=(d, packed))


def run(state):
    stream = torch.cuda.current_stream().cuda_stream
    ws = state["workspace"]
    if "steps" not in state:
        state["plan"].run(state["bindings"], ws.data_ptr(), ws.numel(), stream)
        return state["outputs"]
    state["c"].zero_()                                  # every sequence starts from an empty cell
    hs = state["hs"]
    state["plan"].run_recurrent(state["steps"], state["roles"], state["x"].data_ptr(), state["x_step"], state["h0"].data_ptr(), state["c"].data_ptr(),
                                hs.data_ptr(), hs[0].numel() * hs.element_size(), state["params"], ws.data_ptr(), ws.numel(), stream)
    return [hs, state["c"]]


# ---- how exact the outputs are -------------------------------------------------------------------------------------------
def tolerance(case):
    """About four times the distance of the outputs from their value in 64 bits, as measured.  bf16 layers: that of one rounding
    of the result (2^-9 relative).  A whole network or a recurrence in bf16 rounds after every layer or step.  "max": a single
    element, in units of the result's RMS (or of itself where larger): one more rounding step of bf16 is 2^-8 of it."""
    f, bf16 = case["family"], case["dtype"] == "bf16"
    if f == "resnet18":
        return dict(rel=1.2e-2, max=5e-2) if bf16 else dict(rel=4e-6, max=8e-5)
    if f in ("lenet", "mlp", "lstm"):
        return dict(rel=8e-3, max=4e-2) if bf16 else dict(rel=2e-6, max=4e-5)
    return dict(rel=7e-3, max=2e-2) if bf16 else dict(rel=2.5e-6, max=4e-5)


def _conv64(x, w, stride, pad):
    """conv2d in 64 bits, a matrix product per filter tap."""
    n, c, h, wd = x.shape
    o, _, kh, kw = w.shape
    oh, ow = _out(h, kh, stride, pad), _out(wd, kw, stride, pad)
    xp = torch.nn.functional.pad(x, (pad,) * 4).permute(1, 0, 2, 3)
    y = torch.zeros(o, n * oh * ow, dtype=torch.float64, device=x.device)
    for i in range(kh):
        for j in range(kw):
            tap = xp[:, :, i:i + stride * (oh - 1) + 1:stride, j:j + stride * (ow - 1) + 1:stride].reshape(c, -1).contiguous()
            y += w[:, :, i, j].contiguous() @ tap
    return y.view(o, n, oh, ow).permute(1, 0, 2, 3).contiguous()


def _conv_grad64(dy, x, w, stride, pad):
    n, c, h, wd = x.shape
    o, _, kh, kw = w.shape
    oh, ow = dy.shape[2:]
    xp = torch.nn.functional.pad(x, (pad,) * 4).permute(1, 0, 2, 3)
    dxp, dw = torch.zeros_like(xp), torch.zeros_like(w)
    d = dy.permute(1, 0, 2, 3).reshape(o, -1).contiguous()
    for i in range(kh):
        for j in range(kw):
            at = (slice(None), slice(None), slice(i, i + stride * (oh - 1) + 1, stride), slice(j, j + stride * (ow - 1) + 1, stride))
            dw[:, :, i, j] = d @ xp[at].reshape(c, -1).t().contiguous()
            dxp[at] += (w[:, :, i, j].t().contiguous() @ d).view(c, n, oh, ow)
    return dxp[:, :, pad:pad + h, pad:pad + wd].permute(1, 0, 2, 3).contiguous(), dw


def exact(case, seed):
    f = case["family"]
    d = {k: v.double() for k, v in _data(case, seed).items()}
    ch = lambda b: b.view(1, -1, 1, 1)
    if f == "mlp":
        return [torch.relu(d["x"] @ d["w1"].t() + d["b1"]) @ d["w2"].t() + d["b2"]]
    if f == "dense":
        return [torch.relu(d["x"] @ d["w"].t() + d["b"])]
    if f == "dense_grad":
        return [d["dy"] @ d["w"], d["dy"].t() @ d["x"]]
    if f == "conv":
        return [torch.relu(_conv64(d["x"], d["w"], case["stride"], case["pad"]) + ch(d["b"]) + d.get("r", 0.0))]
    if f == "conv_grad":
        return list(_conv_grad64(d["dy"], d["x"], d["w"], case["stride"], case["pad"]))
    if f == "eltwise":
        return [torch.relu(d["x"] + ch(d["b"]) + d["r"])]
    if f == "lenet":
        y = d["x"]
        for name in ("conv1", "conv2"):
            y = torch.nn.functional.max_pool2d(torch.tanh(_conv64(y, d[name + ".w"], 1, 0) + ch(d[name + ".b"])), 2, 2)
        y = torch.tanh(y.flatten(1) @ d["fc1.w"].t() + d["fc1.b"])
        return [y @ d["fc2.w"].t() + d["fc2.b"]]
    if f == "resnet18":
        y = d["x"]
        for name, _, _, _, s, pad, _, res in _resnet_layers():
            src = skip if name.endswith(".ds") else y1 if res else y
            v = _conv64(src, d[name + ".w"], s, pad) + ch(d[name + ".b"])
            if name == "conv1":
                y = torch.nn.functional.max_pool2d(torch.relu(v), 3, 2, 1)
            elif name.endswith(".ds"):
                skip = v
            elif res:
                y = torch.relu(v + skip)
            else:
                skip, y1 = y, torch.relu(v)
        return [y.mean((2, 3)) @ d["fc.w"].t() + d["fc.b"]]
    m, h = case["batch"], case["hidden"]
    w, b = d["w"].t().contiguous(), d["b"]
    hp, c = torch.zeros(m, h, dtype=torch.float64, device=DEVICE), torch.zeros(m, h, dtype=torch.float64, device=DEVICE)
    hs = []
    for t in range(case["steps"]):
        i, fg, g, o = (torch.cat([d["x"][t], hp], 1) @ w + b).chunk(4, 1)
        c = torch.sigmoid(fg) * c + torch.sigmoid(i) * torch.tanh(g)
        hp = torch.sigmoid(o) * torch.tanh(c)
        hs.append(hp)
    return [torch.stack(hs), c]
