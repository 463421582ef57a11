"""Workloads whose run time is tracked, each one mini-batch through a partition.

A pass is one training step of GPipe's schedule (``runtime.Partition.step``, or
the replay of a step captured with ``capture_step``): M forwards, M
re-materialising backwards, the synchronous update with a nonzero learning
rate, the loss where the partition owns one, and then the bottom layer's
gradients of the tensors named in ``read`` (and of the head's ``read_head``),
fetched with ``gp_get_grad`` into pinned host buffers, as a program does that
watches or exchanges gradients.

The listed cases come from the package's own workloads (``synth.CONFIGS``) at
full width, cut to a few layers so that each is a block of the stack rather
than the whole, plus one whole partition, the fp32 type, and sizes that are
no multiples of the kernels' tiles.
"""
import math

import torch

from paper_1811_06965_amd import gp, runtime
from synth import HEAD_PARAMS, PARAM_IDS, PartitionConfig

BASE = dict(layers=1, d_model=64, d_ff=256, heads=4, seq=32, mem_seq=0, batch=8, micro=4, dtype="bf16",
            kind="encoder", loss="none", vocab=0, label_smoothing=0.0, logit_clip=0.0, optimizer="sgd",
            keep=False, finite=False, graph=False, lr=1e-4, read="ln1_g,wq,wo,w1,b1,w2", read_head="")


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the smallest partition: launches and latency, fp32
        _case("tiny-f32", layers=2, dtype="f32", loss="mse"),
        # fp32 at the width of the small encoder workload, RMSProp
        _case("f32-enc512", layers=2, d_model=512, d_ff=2048, heads=8, seq=128, batch=32, micro=8, dtype="f32",
              loss="mse", optimizer="rmsprop", lr=1e-3),
        # fp32 decoder with its vocabulary head; odd lengths, widths and micro-batch count
        _case("f32-dec-odd", layers=1, d_model=240, d_ff=1000, heads=6, seq=76, mem_seq=52, batch=6, micro=3,
              dtype="f32", kind="decoder", loss="xent_ls", vocab=1000, label_smoothing=0.1, logit_clip=10.0,
              read="ln1_g,wq,wo,xwq,xwk,w1,b1,w2", read_head="lnf_g,wout"),
        # the small encoder workload whole: short sequences, narrow layers
        _case("enc512", layers=8, d_model=512, d_ff=2048, heads=8, seq=128, batch=32, micro=8, loss="mse"),
        # a captured step replayed: launch-bound inner loop of a small model
        _case("enc512-graph", layers=4, d_model=512, d_ff=2048, heads=8, seq=64, batch=32, micro=4, graph=True),
        # ragged: token rows, d_ff and d_model that no tile divides, an odd micro-batch count
        _case("ragged", layers=2, d_model=320, d_ff=1000, heads=5, seq=96, batch=15, micro=5, loss="mse"),
        # stored activations instead of the recompute, checked update, mid-size widths
        _case("stored768", layers=4, d_model=768, d_ff=3072, heads=12, seq=224, batch=24, micro=6, loss="mse",
              optimizer="rmsprop", lr=1e-3, keep=True, finite=True),
        # layers of the d_model 1024 encoder at two of its micro-batch counts
        _case("layer1024-m8", layers=2, d_model=1024, d_ff=8192, heads=16, seq=256, batch=64, micro=8,
              read="ln1_g,wq,wo,w1,b1"),
        _case("layer1024-m32", layers=2, d_model=1024, d_ff=8192, heads=16, seq=256, batch=64, micro=32,
              read="ln1_g,wq,wo,b1,w2"),
        # the last partition of a translation model: decoder layers and the 32000-way head
        _case("dec1024", layers=2, d_model=1024, d_ff=8192, heads=16, seq=256, mem_seq=256, batch=64, micro=16,
              kind="decoder", loss="xent_ls", vocab=32000, label_smoothing=0.1, optimizer="rmsprop", lr=1e-3,
              read="ln1_g,wq,wo,xwq,xwk,b1", read_head="lnf_g,bout"),
        # one layer of the widest encoder
        _case("layer2048", layers=1, d_model=2048, d_ff=16384, heads=32, seq=256, batch=128, micro=32,
              read="ln1_g,wq,wo,b1"),
        # the whole d_model 1024 encoder partition
        _case("enc1024", layers=16, d_model=1024, d_ff=8192, heads=16, seq=256, batch=64, micro=8,
              read="ln1_g,wq,wo,w1,b1"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        c = dict(BASE)
        f32 = rng.random() < 0.3
        dec = rng.random() < 0.35
        c["dtype"] = "f32" if f32 else "bf16"
        c["kind"] = "decoder" if dec else "encoder"
        if f32:
            dh = rng.choice([16, 32, 40, 64])
            c["heads"] = log_int(2, max(2, 512 // dh)) * (2 if dh % 8 else 1)
            c["seq"] = log_int(16, 300)
            c["mem_seq"] = log_int(16, 300) if dec else 0
        else:
            dh = 64
            c["heads"] = log_int(2, 32)
            c["seq"] = 32 * rng.randint(1, 8)
            c["mem_seq"] = 32 * rng.randint(1, 8) if dec else 0
        c["d_model"] = dh * c["heads"]
        c["d_ff"] = max(64, c["d_model"] * rng.choice([2, 3, 4, 8]) - rng.choice([0, 0, 8, 40]))
        c["layers"] = log_int(1, 8)
        c["micro"] = log_int(1, 32)
        c["batch"] = c["micro"] * log_int(1, 16)
        c["loss"] = rng.choice(["none", "mse", "xent_ls"])
        if c["loss"] == "xent_ls":
            c["vocab"] = 8 * log_int(30, 4000)
            c["label_smoothing"] = rng.choice([0.0, 0.1])
            c["logit_clip"] = rng.choice([0.0, 10.0])
            c["read_head"] = "lnf_g,bout"
        if rng.random() < 0.35 and c["loss"] != "none":
            c["optimizer"], c["lr"] = "rmsprop", 1e-3
        c["keep"] = rng.random() < 0.2
        c["finite"] = rng.random() < 0.2
        c["graph"] = rng.random() < 0.2 and not (f32 or dec or c["finite"] or c["keep"]) and c["micro"] > 1
        c["read"] = "ln1_g,wq,wo,b1" + (",xwq,xwk" if dec else "")
        tokens = c["batch"] * max(c["seq"], c["mem_seq"])
        cost = work(c)["flops"] * (10 if f32 else 1)
        n = c["batch"] // c["micro"]
        if f32 and (n * c["seq"] % 4 or n * c["mem_seq"] % 4):
            continue  # fp32 weight gradients take token rows in fours
        if 512 <= tokens <= 32768 and cost <= 1.2e13 and _layer_params(c) * c["layers"] <= 2.0e8:
            return c


# ------------------------------------------------------------------ sizes
def _cfg(case):
    return PartitionConfig("case", layers=case["layers"], d_model=case["d_model"], d_ff=case["d_ff"],
                           heads=case["heads"], seq=case["seq"], batch=case["batch"], micro=case["micro"],
                           dtype=case["dtype"], kind=case["kind"], loss=case["loss"], vocab=case["vocab"],
                           label_smoothing=case["label_smoothing"], mem_seq=case["mem_seq"],
                           optimizer=case["optimizer"], logit_clip=case["logit_clip"])


def _layer_params(case):
    d, f = case["d_model"], case["d_ff"]
    return (8 if case["kind"] == "decoder" else 4) * d * d + 2 * d * f


def work(case):
    """Matrix products of one step (the recompute is the method's: four forward
    passes of work, three with stored activations; the head is not recomputed),
    and every boundary tensor, weight, gradient and optimizer state once."""
    d, f, v = case["d_model"], case["d_ff"], case["vocab"]
    n, s, sm = case["batch"], case["seq"], case["mem_seq"]
    dec = case["kind"] == "decoder"
    t, tm = n * s, n * sm
    fwd = 2.0 * t * (4 * d * d + 2 * d * f) + 4.0 * n * s * s * d * (0.5 if dec else 1.0)
    if dec:
        fwd += 2.0 * t * 2 * d * d + 2.0 * tm * 2 * d * d + 4.0 * n * s * sm * d
    flops = (3 if case["keep"] else 4) * case["layers"] * fwd + 3 * 2.0 * t * d * v
    params = case["layers"] * _layer_params(case) + d * v
    esz = 4 if case["dtype"] == "f32" else 2
    nbytes = params * (12.0 + (8.0 if case["optimizer"] == "rmsprop" else 0.0))
    nbytes += t * d * esz * (4.0 if case["loss"] != "xent_ls" else 3.0) + tm * d * esz * 2.0
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Largest 2-norm difference between two forms of the same step at the same
    # precision.  Measured with other GEMM tiles, split counts and gradient
    # groups: fp32 up to 5e-7 (wide reductions; a drawn size may reach a few
    # times that); bf16 up to 0.027 in gradients and dx, because another order
    # of the fp32 sums moves stored bf16 activations by their last bit and with
    # them a few ReLU masks, which travel through the layers (against 64 bits
    # the same tensors are off by 0.01 to 0.03).
    return {"rel": 1e-5, "max": 4e-3} if case["dtype"] == "f32" else {"rel": 0.03, "max": 0.9}


# ----------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _weights(case, seed):
    """Xavier-uniform matrices, small biases and shifts, gains near one."""
    cfg, g = _cfg(case), _generator(2 * seed)
    bf16 = case["dtype"] == "bf16"

    def one(name, shape):
        if len(shape) == 2:
            w = (torch.rand(shape, generator=g, device="cuda") * 2 - 1) * math.sqrt(6.0 / sum(shape))
        else:
            w = 0.1 * torch.randn(shape, generator=g, device="cuda") + (1.0 if name.endswith("_g") else 0.0)
        return w.bfloat16().float() if bf16 else w

    shapes, head = cfg.param_shapes(), cfg.head_shapes()
    layers = [{p: one(p, shapes[p]) for p in PARAM_IDS if p in shapes} for _ in range(cfg.layers)]
    return layers, {p: one(p, head[p]) for p in HEAD_PARAMS if p in head}


def _inputs(case, seed):
    """Boundary tensors: unit-variance activations and targets, boundary
    gradients of a loss averaged over the tokens, uniform labels."""
    g = _generator(2 * seed + 1)
    t = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    n, s, d = case["batch"], case["seq"], case["d_model"]
    x = torch.randn((n, s, d), generator=g, device="cuda").to(t)
    mem = torch.randn((n, case["mem_seq"], d), generator=g, device="cuda").to(t) if case["mem_seq"] else None
    if case["loss"] == "xent_ls":
        dy = torch.randint(0, case["vocab"], (n, s), generator=g, device="cuda", dtype=torch.int32)
    else:
        dy = torch.randn((n, s, d), generator=g, device="cuda")
        dy = (dy if case["loss"] == "mse" else dy / (n * s)).to(t)
    return x, mem, dy


def _names(text):
    return [p for p in text.split(",") if p]


class State:
    """A configured partition with its weights, one mini-batch of inputs, and
    the output buffers a program reuses from step to step."""

    part = graph = None

    def __init__(self, case, seed):
        self.case = case
        cfg = _cfg(case)
        self.part = runtime.Partition(cfg, check_finite=case["finite"], keep_activations=case["keep"])
        layers, head = _weights(case, seed)
        host = lambda d: {k: v.cpu().numpy() for k, v in d.items()}  # noqa: E731
        self.part.load_params([host(p) for p in layers], host(head))
        self.x, self.mem, self.dy = _inputs(case, seed)
        self.y = torch.empty_like(self.x)
        self.dx = torch.empty_like(self.x)
        self.dmem = torch.empty_like(self.mem) if self.mem is not None else None
        shapes = dict(cfg.param_shapes(), **cfg.head_shapes())
        self.read = {}
        for layer, names in ((0, _names(case["read"])), (-1, _names(case["read_head"]))):
            for p in names:
                buf = torch.empty(shapes[p], dtype=torch.float32, pin_memory=True)
                self.read[p] = (layer, buf, buf.numpy())
        if case["graph"]:
            torch.cuda.synchronize()
            self.graph = self.part.capture_step(self.x, self.mem, self.dy, lr=case["lr"], dx=self.dx,
                                                dmem=self.dmem, want_y=True, y=self.y)

    def __del__(self):
        self.graph = None
        if self.part is not None:
            self.part.close()


def prepare(case, seed):
    return State(case, seed)


def run(state):
    case, out = state.case, {"y": state.y, "dx": state.dx}
    if state.dmem is not None:
        out["dmem"] = state.dmem
    if state.graph is not None:
        state.graph.replay()
    else:
        want_loss = case["loss"] != "none"
        r = state.part.step(state.x, state.mem, state.dy, lr=case["lr"], y=state.y, dx=state.dx, dmem=state.dmem,
                            want_loss=want_loss)
        if want_loss:
            out["loss"] = r["loss"]
    for name, (layer, buf, arr) in state.read.items():
        gp.gp_get_grad(state.part.h, layer, gp.PARAM_ID[name], arr)
        out["grad_" + name] = buf
    return out


# -------------------------------------------------------- 64-bit reference
def _attention(q, k, v, heads, causal):
    n, s, d = q.shape
    dh = d // heads
    split = lambda t: t.reshape(n, -1, heads, dh).transpose(1, 2).contiguous()  # noqa: E731
    q, k, v = split(q), split(k), split(v)
    z = torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dh)
    if causal:
        i = torch.arange(s, device=z.device)
        z = z.masked_fill(i[None, :] > i[:, None], -math.inf)
    return torch.matmul(torch.softmax(z, -1), v).transpose(1, 2).reshape(n, s, d)


def _forward(case, layers, head, x, mem):
    d, h, dec = case["d_model"], case["heads"], case["kind"] == "decoder"
    norm = lambda t, p, k: torch.nn.functional.layer_norm(t, (d,), p[k + "_g"], p[k + "_b"], 1e-5)  # noqa: E731
    for p in layers:
        u = norm(x, p, "ln1")
        a = _attention(u @ p["wq"] + p["bq"], u @ p["wk"] + p["bk"], u @ p["wv"] + p["bv"], h, dec)
        x = x + a @ p["wo"] + p["bo"]
        last = "ln2"
        if dec:
            u = norm(x, p, "ln2")
            a = _attention(u @ p["xwq"] + p["xbq"], mem @ p["xwk"] + p["xbk"], mem @ p["xwv"] + p["xbv"], h, False)
            x = x + a @ p["xwo"] + p["xbo"]
            last = "ln3"
        x = x + torch.relu(norm(x, p, last) @ p["w1"] + p["b1"]) @ p["w2"] + p["b2"]
    return x


def _loss(case, head, y, dy):
    """This chunk's share of the mini-batch loss (for boundary gradients, their product with y)."""
    n, s, d = case["batch"], case["seq"], case["d_model"]
    if case["loss"] == "none":
        return (y * dy).sum()
    if case["loss"] == "mse":
        return (y - dy).square().sum() / (n * s * d)
    h = torch.nn.functional.layer_norm(y, (d,), head["lnf_g"], head["lnf_b"], 1e-5)
    z = h @ head["wout"] + head["bout"]
    if case["logit_clip"] > 0:
        z = z.clamp(-case["logit_clip"], case["logit_clip"])
    return torch.nn.functional.cross_entropy(z.reshape(-1, case["vocab"]), dy.reshape(-1).long(), reduction="sum",
                                             label_smoothing=case["label_smoothing"]) / (n * s)


def exact(case, seed):
    """One step's outputs in 64 bits from the definitions, a few sequences at a time."""
    layers, head = _weights(case, seed)
    wide = lambda d: {k: v.double().requires_grad_() for k, v in d.items()}  # noqa: E731
    layers, head = [wide(p) for p in layers], wide(head)
    x, mem, dy = _inputs(case, seed)
    dy = dy if case["loss"] == "xent_ls" else dy.double()
    chunk = max(1, 2048 // case["seq"])
    ys, dxs, dms, loss = [], [], [], 0.0
    for i in range(0, case["batch"], chunk):
        xi = x[i:i + chunk].double().requires_grad_()
        mi = mem[i:i + chunk].double().requires_grad_() if mem is not None else None
        y = _forward(case, layers, head, xi, mi)
        part = _loss(case, head, y, dy[i:i + chunk])
        part.backward()
        loss += float(part)
        ys.append(y.detach())
        dxs.append(xi.grad)
        if mi is not None:
            dms.append(mi.grad)
    out = {"y": torch.cat(ys), "dx": torch.cat(dxs)}
    if mem is not None:
        out["dmem"] = torch.cat(dms)
    if case["loss"] != "none" and not case["graph"]:
        out["loss"] = loss
    for name in _names(case["read"]):
        out["grad_" + name] = layers[0][name].grad
    for name in _names(case["read_head"]):
        out["grad_" + name] = head[name].grad
    return out
