"""The work whose speed is measured: what a program that trains the network (or part of it) on one GPU calls.

A case is one layer's calls of a training step (forward, backward-data, backward-filter through the entry points that
such a program uses), one glue layer, or a whole step.  `listed()` names the measured ones, `draw()` takes more from
the same ranges, `exact()` gives the results in 64 bits.
"""
import torch
import torch.nn.functional as F

from paper_1312_5853_amd import binding as hp
from paper_1312_5853_amd import stack

# C, H, W, K, R (= S), stride, pad, columns: the layers of the network.  The second layer has two model-parallel
# columns (C and K are the totals).
LAYERS = {
    "conv1": (3, 224, 224, 96, 11, 4, 2, 1),
    "conv2": (96, 27, 27, 256, 5, 1, 2, 2),
    "conv3": (256, 13, 13, 384, 3, 1, 1, 1),
    "conv4": (384, 13, 13, 384, 3, 1, 1, 1),
    "conv5": (384, 13, 13, 256, 3, 1, 1, 1),
}
FC = {"fc6": (9216, 4096), "fc7": (4096, 4096), "fc8": (4096, 1000)}
POOLS = {"pool1": (96, 55, 55), "pool2": (256, 27, 27), "pool5": (256, 13, 13)}


def _conv(N, C, H, W, K, R, stride, pad, cols=1, dtype="f32", relu=False, dx=True):
    """relu: the calls with the ReLU of the layer in them (forward) and the one of the layer below (backward-data)."""
    return dict(kind="conv", N=N, C=C, H=H, W=W, K=K, R=R, stride=stride, pad=pad, cols=cols, dtype=dtype, relu=relu,
                dx=dx)


def _layer(name, N, dtype="f32"):
    C, H, W, K, R, stride, pad, cols = LAYERS[name]
    # the ReLU after the third and fourth layer is applied by the convolution calls; nothing lies below the first layer
    return _conv(N, C, H, W, K, R, stride, pad, cols, dtype, relu=name in ("conv4",), dx=name != "conv1")


def listed():
    cases = [
        # the smallest calls: a 5x5 layer on 32x32 images, four samples; latency and launches count
        dict(_conv(4, 3, 32, 32, 16, 5, 1, 2), name="tiny_f32_n4"),
        # the first layer on a data-parallel shard: forward and backward-filter
        dict(_layer("conv1", 128), name="conv1_f32_n128"),
        # the second layer's two columns
        dict(_layer("conv2", 128), name="conv2_f32_n128"),
        # a small-spatial layer with the ReLUs in its calls, full shard
        dict(_layer("conv4", 128), name="conv4_f32_n128"),
        # a last, ragged mini-batch: odd sample count
        dict(_layer("conv5", 33), name="conv5_f32_n33"),
        # a layer of some other network: odd extents, stride 2, channel counts that fit no tile
        dict(_conv(24, 40, 31, 45, 72, 3, 2, 1), name="odd_f32_n24"),
        # bfloat16 training, the largest mini-batch of one GPU
        dict(_layer("conv3", 256, "bf16"), name="conv3_bf16_n256"),
        # bfloat16, two columns, half a shard
        dict(_layer("conv2", 64, "bf16"), name="conv2_bf16_n64"),
        # ReLU + pooling after the first layer, forward and backward
        dict(kind="pool", planes="pool1", N=128, dtype="f32", name="pool1_f32_n128"),
        # the largest fully connected layer
        dict(kind="fc", N=128, I=9216, O=4096, relu=True, name="fc6_f32_n128"),
        # whole calls: the convolutional stack in bfloat16, and the whole network in fp32 up to its gradients
        dict(kind="stack", N=128, name="stack_bf16_n128"),
        dict(kind="network", N=128, name="network_f32_n128"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "other", "other", "pool", "fc"])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "layer":
        return _layer(rng.choice(sorted(LAYERS)), _log_int(rng, 1, 256), dtype)
    if kind == "other":
        R, stride = rng.choice([1, 3, 3, 5, 7]), rng.choice([1, 1, 1, 2, 3])
        H, W = rng.randint(max(R, 7), 56), rng.randint(max(R, 7), 56)
        C = rng.choice([rng.randint(1, 16), 16 * rng.randint(1, 16), rng.randint(17, 256)])
        K = rng.choice([16 * rng.randint(1, 24), rng.randint(1, 384)])
        # at most 30 GFLOP a pass: below the largest layers of the network
        P, Q = (H + 2 * (R // 2) - R) // stride + 1, (W + 2 * (R // 2) - R) // stride + 1
        most = max(1, min(128, int(30e9 / (2.0 * K * P * Q * C * R * R))))
        return _conv(_log_int(rng, 1, most), C, H, W, K, R, stride, R // 2, 1, dtype, relu=rng.random() < 0.5)
    if kind == "pool":
        return dict(kind="pool", planes=rng.choice(sorted(POOLS)), N=_log_int(rng, 1, 256), dtype=dtype)
    name = rng.choice(sorted(FC) + ["any"])
    I, O = FC[name] if name != "any" else (4 * rng.randint(8, 1024), 4 * rng.randint(2, 1024))
    return dict(kind="fc", N=_log_int(rng, 1, 256), I=I, O=O, relu=rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------------------------
# inputs: activations and gradients N(0, 1), filters N(0, 0.01^2), as the network's own synthetic inputs are
# ---------------------------------------------------------------------------------------------------------------
class _Source:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) % (1 << 62))

    def __call__(self, shape, std=1.0, dtype="f32"):
        t = torch.empty(tuple(shape), dtype=torch.float32, device="cuda").normal_(0.0, std, generator=self.gen)
        return t.to(torch.bfloat16) if dtype == "bf16" else t


def _out(case):
    c = case
    return ((c["H"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["R"]) // c["stride"] + 1)


def _inputs(case, seed):
    c, g = case, _Source(seed)
    if c["kind"] == "conv":
        P, Q = _out(c)
        t = dict(x=g((c["N"], c["C"], c["H"], c["W"]), 1.0, c["dtype"]),
                 w=g((c["K"], c["C"] // c["cols"], c["R"], c["R"]), 0.01, c["dtype"]),
                 dy=g((c["N"], c["K"], P, Q), 1.0, c["dtype"]))
        if c["relu"]:
            t["x"] = torch.relu(t["x"])              # such a layer's input is the output of a ReLU
            t["bias"] = g((c["K"],), 0.1)
        return t
    if c["kind"] == "pool":
        C, H, W = POOLS[c["planes"]]
        return dict(x=g((c["N"], C, H, W), 1.0, c["dtype"]),
                    dy=g((c["N"], C, (H - 3) // 2 + 1, (W - 3) // 2 + 1), 1.0, c["dtype"]))
    if c["kind"] == "fc":
        return dict(x=torch.relu(g((c["N"], c["I"]))), w=g((c["O"], c["I"]), 0.01), bias=g((c["O"],), 0.1),
                    dy=g((c["N"], c["O"])))
    dtype = "bf16" if c["kind"] == "stack" else "f32"
    t = dict(x0=g((c["N"], 3, 224, 224), 1.0, dtype))
    for name in stack.CONV_ORDER:
        C, _, _, K, R, _, _, cols = LAYERS[name]
        t[name] = g((K, C // cols, R, R), 0.01, dtype)
    if c["kind"] == "stack":
        t["g5"] = g((c["N"], 256, 6, 6), 1.0, dtype)
    else:
        for name, (I, O) in FC.items():
            t[name] = g((O, I), 0.01)
            t[name + "_b"] = g((O,), 0.1)
        t["g8"] = g((c["N"], 1000))
    return t


_networks = {}          # one object per (kind, batch size): building its own default inputs on the host takes seconds


def prepare(case, seed):
    c, t = case, _inputs(case, seed)
    if c["kind"] in ("stack", "network"):
        key = (c["kind"], c["N"])
        if key not in _networks:
            _networks[key] = (stack.ConvStack(c["N"], dtype="bf16") if c["kind"] == "stack"
                              else stack.FullNetwork(c["N"]))
        net = _networks[key]
        new = type(net).__new__(type(net))           # the object's buffers of its own, the inputs of this seed
        new.__dict__.update(net.__dict__)
        copy = lambda v: torch.empty_like(v) if isinstance(v, torch.Tensor) else (
            {k: torch.empty_like(u) for k, u in v.items()} if isinstance(v, dict) else v)
        for k, v in net.__dict__.items():
            new.__dict__[k] = copy(v)
        new.ws = hp.Workspace("cuda")
        new.x0 = t["x0"]
        new.w = {n: t[n] for n in stack.CONV_ORDER}
        if c["kind"] == "stack":
            new.g5 = t["g5"]
        else:
            new.fc_w = {n: t[n] for n in FC}
            new.fc_b = {n: t[n + "_b"] for n in FC}
            new.g8 = t["g8"]
            new.params, new.vel = [], []
        return dict(case=c, net=new)
    s = dict(t, case=c, ws=hp.Workspace("cuda"))
    if c["kind"] == "conv":
        # activations and input gradients have the element type of the inputs, filter gradients are fp32
        s["y"] = torch.empty_like(t["dy"])
        s["dx"] = torch.empty_like(t["x"])
        s["dw"] = torch.empty(t["w"].shape, dtype=torch.float32, device="cuda")
    elif c["kind"] == "pool":
        s["y"], s["dx"] = torch.empty_like(t["dy"]), torch.empty_like(t["x"])
    else:
        s["y"], s["dx"], s["dw"] = torch.empty_like(t["dy"]), torch.empty_like(t["x"]), torch.empty_like(t["w"])
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "stack":
        net = s["net"]
        a5 = net.forward()
        dw = net.backward()
        return [a5] + [dw[n] for n in stack.CONV_ORDER]
    if c["kind"] == "network":
        net = s["net"]
        logits = net.forward()
        net.backward()
        return ([logits] + [net.dw[n] for n in stack.CONV_ORDER] + [net.fc_dw[n] for n in FC]
                + [net.fc_db[n] for n in FC])
    x, dy, ws = s["x"], s["dy"], s.get("ws")
    if c["kind"] == "pool":
        hp.relu_maxpool3x3s2_fwd(x, s["y"])
        hp.relu_maxpool3x3s2_bwd(x, dy, s["dx"])
        return [s["y"], s["dx"]]
    w = s["w"]
    if c["kind"] == "fc":
        hp.fc_fwd(x, w, s["bias"], relu=c["relu"], y=s["y"], ws=ws)
        hp.fc_bwd_filter(x, dy, dw=s["dw"], ws=ws)
        hp.fc_bwd_data(dy, w, dx=s["dx"], ws=ws)
        return [s["y"], s["dw"], s["dx"]]
    st, pad, R = c["stride"], c["pad"], c["R"]
    if c["cols"] > 1:
        hp.conv_fwd_grouped(x, w, st, pad, c["cols"], y=s["y"], ws=ws)
        hp.conv_bwd_filter_grouped(x, dy, R, R, st, pad, c["cols"], dw=s["dw"], ws=ws)
        hp.conv_bwd_data_grouped(dy, w, c["H"], c["W"], st, pad, c["cols"], dx=s["dx"], ws=ws)
    elif c["relu"]:
        hp.conv_fwd_bias_relu(x, w, s["bias"], st, pad, y=s["y"], ws=ws)
        hp.conv_bwd_filter(x, dy, R, R, st, pad, dw=s["dw"], ws=ws)
        hp.conv_bwd_data_relu(dy, w, x, st, pad, dx=s["dx"], ws=ws)
    else:
        hp.conv_fwd(x, w, st, pad, y=s["y"], ws=ws)
        hp.conv_bwd_filter(x, dy, R, R, st, pad, dw=s["dw"], ws=ws)
        if c["dx"]:
            hp.conv_bwd_data(dy, w, c["H"], c["W"], st, pad, dx=s["dx"], ws=ws)
    return [s["y"], s["dw"], s["dx"]] if c["dx"] else [s["y"], s["dw"]]


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------
def _work_parts(case):
    c = case
    if c["kind"] == "conv":
        P, Q = _out(c)
        eb = 2 if c["dtype"] == "bf16" else 4
        x, y = c["N"] * c["C"] * c["H"] * c["W"], c["N"] * c["K"] * P * Q
        w = c["K"] * (c["C"] // c["cols"]) * c["R"] ** 2
        passes = 3 if c["dx"] else 2
        # x and dy serve two calls each but are read once at least; y, dx and dw (fp32) are written once
        bytes_ = eb * (x + w + 2 * y) + 4 * w + (eb * x if c["dx"] else 0)
        return bytes_, passes * 2.0 * y * w / c["K"]
    if c["kind"] == "pool":
        C, H, W = POOLS[c["planes"]]
        eb = 2 if c["dtype"] == "bf16" else 4
        x, y = c["N"] * C * H * W, c["N"] * C * ((H - 3) // 2 + 1) * ((W - 3) // 2 + 1)
        return eb * (2 * x + 2 * y), 10.0 * y
    if c["kind"] == "fc":
        N, I, O = c["N"], c["I"], c["O"]
        return 4 * (2 * N * I + 2 * N * O + 2 * I * O + O), 6.0 * N * I * O
    raise ValueError(c["kind"])


def work(case):
    c = case
    if c["kind"] in ("conv", "pool", "fc"):
        b, f = _work_parts(c)
        return {"bytes": float(b), "flops": float(f)}
    dtype = "bf16" if c["kind"] == "stack" else "f32"
    parts = [_work_parts(_layer(n, c["N"], dtype)) for n in stack.CONV_ORDER]
    parts += [_work_parts(dict(kind="pool", planes=p, N=c["N"], dtype=dtype)) for p in POOLS]
    if c["kind"] == "network":
        parts += [_work_parts(dict(kind="fc", N=c["N"], I=I, O=O)) for I, O in FC.values()]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


# About four times the largest relative error against `exact` that was measured over the listed cases and draws.
def tolerance(case):
    c = case
    if c["kind"] == "stack":
        return {"rel": 0.2}           # roundings between the layers, pooling windows whose two largest values swap (5.7e-2)
    if c["kind"] == "network":
        return {"rel": 2e-2}          # pooling windows whose two largest values are closer than the error of a sum (5.6e-3)
    if c.get("dtype") == "bf16":
        return {"rel": 7e-3}           # each result rounded once to 8 bits (1.7e-3)
    if c["kind"] == "pool":
        return {"rel": 1e-7}           # maxima are input values; sums of at most four gradients (2.5e-8)
    if c["kind"] == "fc":
        return {"rel": 2e-6}           # fp32 sums of up to 9216 products (4.4e-7)
    return {"rel": 5e-6}               # fp32 sums of up to 9408 products forward, 4e5 positions in dw (1.1e-6)


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits, from the definitions (patches as a matrix, a few samples at a time)
# ---------------------------------------------------------------------------------------------------------------
def _chunks(N, per_sample):
    step = max(1, int(2.0e8 / per_sample))
    return [(i, min(N, i + step)) for i in range(0, N, step)]


def _conv64(x, w, stride, pad):
    K, C, R, S = w.shape
    N, _, H, W = x.shape
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    y = torch.empty((N, K, P, Q), dtype=torch.float64, device=x.device)
    for a, b in _chunks(N, C * R * S * P * Q):
        cols = F.unfold(x[a:b].double(), (R, S), padding=pad, stride=stride)
        y[a:b] = torch.matmul(w.double().reshape(K, -1), cols).reshape(b - a, K, P, Q)
    return y


def _conv64_dx(dy, w, H, W, stride, pad):
    K, C, R, S = w.shape
    N, _, P, Q = dy.shape
    dx = torch.empty((N, C, H, W), dtype=torch.float64, device=dy.device)
    wt = w.double().reshape(K, -1).t().contiguous()
    for a, b in _chunks(N, C * R * S * P * Q):
        cols = torch.matmul(wt, dy[a:b].double().reshape(b - a, K, P * Q))
        dx[a:b] = F.fold(cols, (H, W), (R, S), padding=pad, stride=stride)
    return dx


def _conv64_dw(x, dy, R, S, stride, pad):
    N, C = x.shape[:2]
    K, PQ = dy.shape[1], dy.shape[2] * dy.shape[3]
    dw = torch.zeros((K, C * R * S), dtype=torch.float64, device=x.device)
    for a, b in _chunks(N, C * R * S * PQ):
        cols = F.unfold(x[a:b].double(), (R, S), padding=pad, stride=stride).transpose(0, 1).reshape(C * R * S, -1)
        dw += dy[a:b].double().reshape(b - a, K, PQ).transpose(0, 1).reshape(K, -1) @ cols.t().contiguous()
    return dw.reshape(K, C, R, S)


def _columns(fn, cols, a, b, dim_a, dim_b, dim_out):
    parts = [fn(u, v) for u, v in zip(a.chunk(cols, dim_a), b.chunk(cols, dim_b))]
    return parts[0] if cols == 1 else torch.cat(parts, dim_out)


def _pool64_bwd(pre, dy):
    """Gradient of relu followed by 3x3/2 max pooling: to the first maximum of each window, where it is positive."""
    y, idx = F.max_pool2d(pre.double(), 3, 2, return_indices=True)
    N, C, H, W = pre.shape
    dx = torch.zeros((N, C, H * W), dtype=torch.float64, device=pre.device)
    g = torch.where(y > 0, dy.double(), torch.zeros((), dtype=torch.float64, device=pre.device))
    dx.scatter_add_(2, idx.reshape(N, C, -1), g.reshape(N, C, -1))
    return dx.reshape(N, C, H, W)


def _round_bf16(v):
    return v.to(torch.float32).to(torch.bfloat16).double()


def _exact_network(t, bf16=False):
    """Forward and backward of the convolutional layers and, where its weights are there, of the fully connected ones.
    bf16: every activation and gradient that the network stores is rounded to bfloat16, the filter gradients are not."""
    keep = _round_bf16 if bf16 else (lambda v: v)
    x, ins, pre = t["x0"], {}, {}
    for name in stack.CONV_ORDER:
        _, _, _, _, _, st, pad, cols = LAYERS[name]
        ins[name] = x
        pre[name] = keep(_columns(lambda u, v: _conv64(u, v, st, pad), cols, x, t[name], 1, 0, 1))
        x = torch.relu(pre[name])
        if name in ("conv1", "conv2", "conv5"):
            x = F.max_pool2d(x, 3, 2)
    if "g5" in t:
        top, d, fdw, fdb = [x], t["g5"].double(), {}, {}
    else:
        a, acts = x.reshape(x.shape[0], -1), []
        for name in FC:
            acts.append(a)
            a = a @ t[name].double().t() + t[name + "_b"].double()
            if name != "fc8":
                a = torch.relu(a)
        top, d, fdw, fdb = [a], t["g8"].double(), {}, {}
        for i, name in reversed(list(enumerate(FC))):
            if name != "fc8":
                d = d * (acts[i + 1] > 0)
            fdw[name], fdb[name] = d.t() @ acts[i], d.sum(0)
            d = d @ t[name].double()
        d = d.reshape(x.shape)
    dw = {}
    for name in reversed(stack.CONV_ORDER):
        _, H, W, _, R, st, pad, cols = LAYERS[name]
        d = keep(_pool64_bwd(pre[name], d)) if name in ("conv1", "conv2", "conv5") else d * (pre[name] > 0)
        dw[name] = _columns(lambda u, v: _conv64_dw(u, v, R, R, st, pad), cols, ins[name], d, 1, 1, 0)
        if name != "conv1":
            d = keep(_columns(lambda u, v: _conv64_dx(u, v, H, W, st, pad), cols, d, t[name], 1, 0, 1))
    return top + [dw[n] for n in stack.CONV_ORDER] + [fdw[n] for n in fdw and FC] + [fdb[n] for n in fdb and FC]


def exact(case, seed):
    c = case
    t = _inputs(c, seed)
    if c["kind"] in ("stack", "network"):
        return _exact_network(t, bf16=c["kind"] == "stack")
    if c["kind"] == "pool":
        return [F.max_pool2d(torch.relu(t["x"].double()), 3, 2), _pool64_bwd(t["x"], t["dy"])]
    if c["kind"] == "fc":
        x, w, dy = t["x"].double(), t["w"].double(), t["dy"].double()
        y = x @ w.t() + t["bias"].double()
        return [torch.relu(y) if c["relu"] else y, dy.t() @ x, dy @ w]
    st, pad, R, cols = c["stride"], c["pad"], c["R"], c["cols"]
    y = _columns(lambda u, v: _conv64(u, v, st, pad), cols, t["x"], t["w"], 1, 0, 1)
    dw = _columns(lambda u, v: _conv64_dw(u, v, R, R, st, pad), cols, t["x"], t["dy"], 1, 1, 0)
    if c["relu"]:
        y = torch.relu(y + t["bias"].double().reshape(1, -1, 1, 1))
    if not c["dx"]:
        return [y, dw]
    dx = _columns(lambda u, v: _conv64_dx(u, v, c["H"], c["W"], st, pad), cols, t["dy"], t["w"], 1, 0, 1)
    if c["relu"]:
        dx = dx * (t["x"] > 0)
    return [y, dw, dx]
