"""The workloads this library is timed on, through its public entry points.

Four kinds of work: a chain of fully-connected layers (a training step, or forward only), one convolution layer's
training step, a small convolution | flatten | fully-connected network's training step, and a tiling conversion of one
tensor.  `listed()` names the workloads; `draw()` gives further sizes from the same ranges.

What a user's program has in hand before a step - the plan, the shards of its tensors, one workspace - is made by
`prepare()`; `run()` is one step.  Shards are cut from the full tensor, so replicas hold equal values.
"""
import functools
import math

import torch

import paper_1805_04170_amd as tt

DEVICE = "cuda:0"


def listed():
    return [
        # A small fp32 chain, all of it launch latency: what debugging runs and small heads on a larger model cost.
        dict(name="tiny_mlp_f32", kind="fc", mode="step", dtype="f32", batch=32, widths="256-512-256-10", k=2,
             tiling="planner", w_std=0.02),
        # AlexNet's classifier, one training step over 8 shards.
        dict(name="alexnet_fc", kind="fc", mode="step", dtype="bf16", batch=256, widths="9216-4096-4096-1000", k=3,
             tiling="planner", w_std=0.01),
        # VGG-16's classifier, one training step over 8 shards (the benchmark's headline workload).
        dict(name="vgg16_fc", kind="fc", mode="step", dtype="bf16", batch=256, widths="25088-4096-4096-1000", k=3,
             tiling="planner", w_std=0.005),
        # AlexNet's classifier answering a small batch: forward only, weights streamed once.
        dict(name="alexnet_fc_serve16", kind="fc", mode="forward", dtype="bf16", batch=16, widths="9216-4096-4096-1000",
             k=3, tiling="planner", w_std=0.01),
        # Layer widths that are no round numbers: shards whose rows are not whole 16-byte vectors.
        dict(name="ragged_mlp", kind="fc", mode="step", dtype="bf16", batch=100, widths="1500-900-300-20", k=2,
             tiling="planner", w_std=0.03),
        # Wide layers under a forced 4 x 4 grid of every tensor (16 shards): partial sums and conversions at each layer.
        dict(name="wide_mlp_grid", kind="fc", mode="step", dtype="bf16", batch=512, widths="8192-8192-8192-8192-8192", k=4,
             tiling="grid", w_std=0.01),
        # The same layers with all four cuts on the reduction dimension: 16 partial sums per result.
        dict(name="wide_mlp_f3", kind="fc", mode="step", dtype="bf16", batch=512, widths="8192-8192-8192-8192-8192", k=4,
             tiling="f3", w_std=0.01),
        # Large batch, nothing cut: bound by arithmetic alone.
        dict(name="mlp_8k_untiled", kind="fc", mode="step", dtype="bf16", batch=2048, widths="8192-8192-8192-8192-8192", k=0,
             tiling="planner", w_std=0.01),
        # VGG-16's conv4 layer as the planner cuts it, and as data parallelism would.
        dict(name="vgg16_conv4_planner", kind="conv", N=64, C=512, K=512, H=28, W=28, R=3, pad=1, k=3, split="planner"),
        dict(name="vgg16_conv4_batch", kind="conv", N=64, C=512, K=512, H=28, W=28, R=3, pad=1, k=3, split="batch"),
        # A small network: convolution, flatten, classifier.
        dict(name="conv_flatten_fc", kind="net", N=32, C=64, K=64, H=14, W=14, widths="512-256-32", k=3),
        # The first VGG-16 classifier weight going from row blocks to column blocks.
        dict(name="retile_w1", kind="retile", rows=25088, cols=4096, elem=2, A="RRR", B="CCC"),
    ]


# ------------------------------------------------------------------------------------------------- further cases

def _log_int(rng, lo, hi, step):
    """an integer between lo and hi, spread over the logarithm, a multiple of step"""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


def draw(rng):
    kind = rng.choice(["fc", "fc", "fc", "fc_ragged", "fc_f32", "fc_forward", "conv", "conv", "net", "retile"])
    if kind in ("fc", "fc_ragged", "fc_f32", "fc_forward"):
        while True:
            k = rng.randint(0, 2 if kind == "fc_f32" else 3)
            n = 1 << k
            layers = rng.randint(1, 4)
            if kind == "fc":
                batch, step, lo, hi, cap = _log_int(rng, 32, 2048, n), 8 * n, 512, 16384, 2.0e12
            elif kind == "fc_forward":
                batch, step, lo, hi, cap = _log_int(rng, 8, 256, n), 8 * n, 512, 12288, 1.0e12
            elif kind == "fc_ragged":
                batch, step, lo, hi, cap = _log_int(rng, 16, 256, n), n, 20, 2048, 2.0e10
            else:
                batch, step, lo, hi, cap = _log_int(rng, 8, 256, n), n, 16, 1024, 5.0e9
            widths = [_log_int(rng, lo, hi, step) for _ in range(layers + 1)]
            weights = sum(a * b for a, b in zip(widths, widths[1:]))
            if 6.0 * batch * weights > cap or weights > 270e6:
                continue
            return dict(kind="fc", mode="forward" if kind == "fc_forward" else "step",
                        dtype="f32" if kind == "fc_f32" else "bf16", batch=batch, widths="-".join(map(str, widths)), k=k,
                        tiling="planner", w_std=round(1.0 / math.sqrt(sum(widths[:-1]) / layers), 4))
    if kind == "conv":
        while True:
            k = rng.randint(0, 3)
            n = 1 << k
            R = rng.choice([1, 3, 3])
            c = dict(kind="conv", N=_log_int(rng, 8, 128, n), C=_log_int(rng, 64, 512, 8 * n), K=_log_int(rng, 64, 512, 8 * n),
                     H=rng.randint(7, 56), W=rng.randint(7, 56), R=R, pad=R // 2, k=k,
                     split=rng.choice(["planner", "batch", "out_channel"]))
            pixels = c["N"] * c["H"] * c["W"]
            if 6.0 * pixels * c["C"] * c["K"] * R * R < 7.2e11 and pixels * max(c["C"], c["K"]) < 6e7:
                return c
    if kind == "net":
        k = rng.randint(1, 3)
        n = 1 << k
        return dict(kind="net", N=_log_int(rng, 16, 64, n), C=8 * n * rng.randint(1, 2), K=8 * n * rng.randint(1, 2),
                    H=rng.randint(6, 14), W=rng.randint(6, 14),
                    widths="-".join(str(_log_int(rng, 32, 1024, 8 * n)) for _ in range(rng.randint(1, 3))), k=k)
    while True:
        k = rng.randint(1, 3)
        A, B = ("".join(rng.choice("RRCCr") for _ in range(k)) for _ in range(2))
        step = (1 << k) * rng.choice([1, 8])
        c = dict(kind="retile", rows=_log_int(rng, 64, 32768, 1 << k), cols=_log_int(rng, 64, 32768, step),
                 elem=rng.choice([2, 4]), A=A, B=B)
        if c["rows"] * c["cols"] * c["elem"] * (1 << B.count("r")) < 2.2e8:
            return c


# -------------------------------------------------------------------------------------------------------- tensors

class _Maker:
    """Seeded normal tensors on the GPU, as the 2^k shards of a tiling."""

    def __init__(self, seed):
        self.gen = torch.Generator(device=DEVICE)
        self.gen.manual_seed(seed)

    def normal(self, rows, cols, t, std, dtype):
        full = torch.empty((rows, cols), dtype=torch.float32, device=DEVICE)
        full.normal_(0.0, std, generator=self.gen)
        return _cut(full.to(dtype), t)


def _block_of(t, s):
    """(row block, column block) that shard s of tiling t holds"""
    k, rb, cb = len(t), 0, 0
    for j, ch in enumerate(t):
        bit = (s >> (k - 1 - j)) & 1
        if ch == "R":
            rb = 2 * rb + bit
        elif ch == "C":
            cb = 2 * cb + bit
    return rb, cb


def _cut(full, t):
    sr, sc = tt.tt_shard_shape(full.shape[0], full.shape[1], t)
    out = []
    for s in range(1 << len(t)):
        rb, cb = _block_of(t, s)
        out.append(full[rb * sr:(rb + 1) * sr, cb * sc:(cb + 1) * sc].clone(memory_format=torch.contiguous_format))
    return out


class _Shards(list):
    """The shards of a result, cut from one buffer (`whole`) at 256-byte boundaries."""


def _empty(rows, cols, t, dtype):
    sr, sc = tt.tt_shard_shape(rows, cols, t)
    n, unit = 1 << len(t), 256 // torch.empty(0, dtype=dtype).element_size()
    pitch = -(-sr * sc // unit) * unit
    whole = torch.zeros(n * pitch, dtype=dtype, device=DEVICE)
    out = _Shards(whole[s * pitch:s * pitch + sr * sc].view(sr, sc) for s in range(n))
    out.whole = whole
    return out


def _workspace(nbytes):
    return torch.empty(max(256, nbytes), dtype=torch.uint8, device=DEVICE)


def _widths(case):
    return [int(w) for w in case["widths"].split("-")]


def _torch_dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _swap(t):
    """letters of a filter's tiling on its (K*R*S) x C storage matrix"""
    return t.translate(str.maketrans("RC", "CR"))


# ---------------------------------------------------------------------------------------------------------- plans

@functools.lru_cache(maxsize=64)
def _fc_plan(widths, batch, k, tiling):
    """tilings x[0..L], g[0..L], w[1..L] and the three form sequences of every layer"""
    L = len(widths) - 1
    if tiling == "grid":    # every tensor a 4 x 4 grid; forward and data gradient cut the reduction dimension twice
        return ["RRCC"] * (L + 1), ["RRCC"] * (L + 1), ["RRCC"] * L, [["3322", "2233", "1122"]] * L
    if tiling == "f3":      # all four cuts on the forward product's reduction dimension
        return ["CCCC"] * (L + 1), ["rrrr"] * (L + 1), ["RRRR"] * L, [["3333", "2222", "1111"]] * L
    p = tt.tt_plan_chain([tt.layer("fc", "none", a, b) for a, b in zip(widths, widths[1:])], batch, k)
    return p.x(), p.g(), p.w(), [[p.forms(l, op) for op in range(3)] for l in range(1, L + 1)]


class _FcChain:
    """A chain of fully-connected layers (ReLU after every layer but the last) under a plan."""

    def __init__(self, case, seed):
        w = self.w = _widths(case)
        self.b, self.k, self.dt = case["batch"], case["k"], case["dtype"]
        self.L = len(w) - 1
        self.backward = case["mode"] == "step"
        dt, make = _torch_dtype(self.dt), _Maker(seed)
        self.tx, self.tg, self.tw, self.f = _fc_plan(tuple(w), self.b, self.k, case["tiling"])
        self.lay = [tt.layer("fc", "relu" if l < self.L else "none", w[l - 1], w[l]) for l in range(1, self.L + 1)]
        self.x = [make.normal(self.b, w[0], self.tx[0], 1.0, dt)]
        self.x += [_empty(self.b, w[l], self.tx[l], dt) for l in range(1, self.L + 1)]
        self.W = [make.normal(w[l - 1], w[l], self.tw[l - 1], case["w_std"], dt) for l in range(1, self.L + 1)]
        need = [self._need(l, tt.TT_OP_FWD) for l in range(1, self.L + 1)]
        # what fits the library's own scratch array needs no workspace for its forward pass
        self.static = not self.backward and max(need) <= tt.TT_STATIC_SCRATCH_BYTES
        if self.backward:
            self.g = [_empty(self.b, w[l], self.tg[l], dt) for l in range(self.L)]
            self.g.append(make.normal(self.b, w[self.L], self.tg[self.L], 1.0, dt))
            self.dW = [_empty(w[l - 1], w[l], self.tw[l - 1], dt) for l in range(1, self.L + 1)]
            need += [self._need(l, tt.TT_OP_DGRAD) for l in range(1, self.L + 1)]
        self.ws = None if self.static else _workspace(max(need))

    def _need(self, l, op):
        f = self.f[l - 1]
        lay, t = self.lay[l - 1], (self.tx[l - 1], self.tw[l - 1], self.tx[l])
        if op == tt.TT_OP_FWD:
            return tt.tt_fc_workspace_bytes(lay, self.b, self.k, self.dt, op, *t, forms_a=f[0])
        return tt.tt_fc_workspace_bytes(lay, self.b, self.k, self.dt, op, *t, self.tg[l], self.tg[l - 1], f[1], f[2])

    def forward_layers(self):
        for l in range(1, self.L + 1):
            a = (self.lay[l - 1], self.b, self.k, self.dt, self.tx[l - 1], self.tw[l - 1], self.tx[l], self.f[l - 1][0],
                 self.x[l - 1], self.W[l - 1], self.x[l])
            if self.static:
                tt.tt_fc_forward_static(*a)
            else:
                tt.tt_fc_forward(*a, self.ws)

    def backward_layers(self):
        for l in range(self.L, 0, -1):
            tt.tt_fc_backward(self.lay[l - 1], self.b, self.k, self.dt, self.tx[l - 1], self.tw[l - 1], self.tx[l],
                              self.tg[l], self.tg[l - 1], self.f[l - 1][1], self.f[l - 1][2], self.x[l - 1], self.W[l - 1],
                              self.x[l], self.g[l], self.g[l - 1], self.dW[l - 1], self.ws)

    def step(self):
        self.forward_layers()
        if not self.backward:
            return dict(x=[x.whole for x in self.x[1:]])
        self.backward_layers()
        return dict(y=self.x[self.L].whole, dW=[d.whole for d in self.dW], dX=self.g[0].whole)


def _conv_layer(case):
    return tt.layer("conv", "none", case["C"], case["K"], H=case["H"], W=case["W"], R=case["R"], S=case["R"], pad=case["pad"])


def _conv_plan(case):
    """tilings of X, W, Y, dY, dX and the three form sequences"""
    k = case["k"]
    if case["split"] == "planner":
        p = tt.tt_plan_chain([_conv_layer(case)], case["N"], k)
        return (p.x()[0], p.w()[0], p.x()[1], p.g()[1], p.g()[0]), [p.forms(1, op) for op in range(3)]
    if case["split"] == "batch":
        return ("R" * k, "r" * k, "R" * k, "R" * k, "R" * k), ["1" * k, "1" * k, "3" * k]
    return ("r" * k, "C" * k, "C" * k, "C" * k, "r" * k), ["2" * k, "3" * k, "2" * k]


class _Conv:
    """One convolution layer's training step."""

    def __init__(self, case, seed):
        N, C, K, H, W, R, pad = (case[n] for n in ("N", "C", "K", "H", "W", "R", "pad"))
        k = self.k = case["k"]
        self.N = N
        P, Q = H + 2 * pad - R + 1, W + 2 * pad - R + 1
        self.lay = _conv_layer(case)
        self.t, self.f = _conv_plan(case)
        tX, tW, tY, tdY, tdX = self.t
        bf, make = torch.bfloat16, _Maker(seed)
        self.X = make.normal(N * H * W, C, tX, 1.0, bf)
        self.W = make.normal(K * R * R, C, _swap(tW), 0.02, bf)
        self.dY = make.normal(N * P * Q, K, tdY, 1.0, bf)
        self.Y = _empty(N * P * Q, K, tY, bf)
        self.dX = _empty(N * H * W, C, tdX, bf)
        self.dW = _empty(K * R * R, C, _swap(tW), bf)
        self.ws = _workspace(max(
            tt.tt_conv_workspace_bytes(self.lay, N, k, "bf16", tt.TT_OP_FWD, tX, tW, tY, forms_a=self.f[0]),
            tt.tt_conv_workspace_bytes(self.lay, N, k, "bf16", tt.TT_OP_DGRAD, tX, tW, tY, tdY, tdX, self.f[1], self.f[2])))

    def step(self):
        tX, tW, tY, tdY, tdX = self.t
        tt.tt_conv_forward(self.lay, self.N, self.k, "bf16", tX, tW, tY, self.f[0], self.X, self.W, self.Y, self.ws)
        tt.tt_conv_backward(self.lay, self.N, self.k, "bf16", tX, tW, tY, tdY, tdX, self.f[1], self.f[2], self.X, self.W,
                            self.Y, self.dY, self.dX, self.dW, self.ws)
        return dict(y=self.Y.whole, dW=self.dW.whole, dX=self.dX.whole)


def _net_plan(case):
    """the convolution, the fully-connected layers, the plan of the chain"""
    conv = tt.layer("conv", "relu", case["C"], case["K"], H=case["H"], W=case["W"], R=3, S=3, pad=1)
    dims = [case["K"] * case["H"] * case["W"]] + _widths(case)
    n = len(dims) - 1
    fcs = [tt.layer("fc", "relu" if i + 1 < n else "none", dims[i], dims[i + 1]) for i in range(n)]
    return conv, fcs, tt.tt_plan_chain([conv] + fcs, case["N"], case["k"])


class _Net:
    """3 x 3 convolution (ReLU) | flatten | fully-connected layers (ReLU between), the whole chain under one plan."""

    def __init__(self, case, seed):
        N, C, K, H, W, k = (case[n] for n in ("N", "C", "K", "H", "W", "k"))
        self.N, self.C, self.K, self.HW, self.k = N, C, K, H * W, k
        dims = self.dims = [K * H * W] + _widths(case)
        n = len(dims) - 1
        conv, self.fcs, p = _net_plan(case)
        self.conv = conv
        tx, tg, tw = self.tx, self.tg, self.tw = p.x(), p.g(), p.w()
        f = self.f = [[p.forms(l, op) for op in range(3)] for l in range(1, n + 2)]
        bf, make = torch.bfloat16, _Maker(seed)
        self.x0 = make.normal(N * H * W, C, tx[0], 1.0, bf)
        self.Wc = make.normal(K * 9, C, _swap(tw[0]), 1.5 / math.sqrt(9 * C), bf)
        self.Wf = [make.normal(dims[i], dims[i + 1], tw[1 + i], 1.5 / math.sqrt(dims[i]), bf) for i in range(n)]
        self.y1 = _empty(N * H * W, K, tx[1], bf)
        self.acts = [_empty(N, dims[i], tx[1 + i], bf) for i in range(n + 1)]
        self.gs = [_empty(N, dims[i], tg[1 + i], bf) for i in range(n)] + [make.normal(N, dims[n], tg[1 + n], 1.0, bf)]
        self.dWf = [_empty(dims[i], dims[i + 1], tw[1 + i], bf) for i in range(n)]
        self.dy1 = _empty(N * H * W, K, tg[1], bf)
        self.dx0 = _empty(N * H * W, C, tg[0], bf)
        self.dWc = _empty(K * 9, C, _swap(tw[0]), bf)
        need = [tt.tt_conv_workspace_bytes(conv, N, k, "bf16", tt.TT_OP_FWD, tx[0], tw[0], tx[1], forms_a=f[0][0]),
                tt.tt_conv_workspace_bytes(conv, N, k, "bf16", tt.TT_OP_DGRAD, tx[0], tw[0], tx[1], tg[1], tg[0], f[0][1], f[0][2])]
        for i, lay in enumerate(self.fcs):
            l = 1 + i
            need.append(tt.tt_fc_workspace_bytes(lay, N, k, "bf16", tt.TT_OP_FWD, tx[l], tw[l], tx[l + 1], forms_a=f[l][0]))
            need.append(tt.tt_fc_workspace_bytes(lay, N, k, "bf16", tt.TT_OP_DGRAD, tx[l], tw[l], tx[l + 1], tg[l + 1], tg[l],
                                                 f[l][1], f[l][2]))
        self.ws = _workspace(max(need))

    def step(self):
        N, k, tx, tg, tw, f, ws = self.N, self.k, self.tx, self.tg, self.tw, self.f, self.ws
        tt.tt_conv_forward(self.conv, N, k, "bf16", tx[0], tw[0], tx[1], f[0][0], self.x0, self.Wc, self.y1, ws)
        tt.tt_flatten(self.acts[0], tx[1], self.y1, tx[1], N, self.K, self.HW, 2, True, k=k)
        for i, lay in enumerate(self.fcs):
            tt.tt_fc_forward(lay, N, k, "bf16", tx[1 + i], tw[1 + i], tx[2 + i], f[1 + i][0], self.acts[i], self.Wf[i],
                             self.acts[i + 1], ws)
        for i in reversed(range(len(self.fcs))):
            l = 1 + i
            tt.tt_fc_backward(self.fcs[i], N, k, "bf16", tx[l], tw[l], tx[l + 1], tg[l + 1], tg[l], f[l][1], f[l][2],
                              self.acts[i], self.Wf[i], self.acts[i + 1], self.gs[i + 1], self.gs[i], self.dWf[i], ws)
        tt.tt_flatten(self.dy1, tg[1], self.gs[0], tg[1], N, self.K, self.HW, 2, False, k=k)
        tt.tt_conv_backward(self.conv, N, k, "bf16", tx[0], tw[0], tx[1], tg[1], tg[0], f[0][1], f[0][2], self.x0, self.Wc,
                            self.y1, self.dy1, self.dx0, self.dWc, ws)
        return dict(y=self.acts[-1].whole, dWf=[d.whole for d in self.dWf], dWc=self.dWc.whole, dX=self.dx0.whole)


class _Retile:
    def __init__(self, case, seed):
        self.rows, self.cols, self.elem, self.A, self.B = (case[n] for n in ("rows", "cols", "elem", "A", "B"))
        dt = torch.bfloat16 if self.elem == 2 else torch.float32
        self.src = _Maker(seed).normal(self.rows, self.cols, self.A, 1.0, dt)
        self.dst = _empty(self.rows, self.cols, self.B, dt)

    def step(self):
        tt.tt_retile(self.dst, self.B, self.src, self.A, self.rows, self.cols, self.elem)
        return self.dst.whole


def prepare(case, seed):
    return dict(fc=_FcChain, conv=_Conv, net=_Net, retile=_Retile)[case["kind"]](case, seed)


def run(state):
    return state.step()


# ------------------------------------------------------------------------------------------------ work, tolerance

def work(case):
    """Inputs and weights read once, results and gradients written once (every tensor counted without its replicas)."""
    kind = case["kind"]
    if kind == "retile":
        one = case["rows"] * case["cols"] * case["elem"]
        return dict(bytes=one * (1 + (1 << case["B"].count("r"))), flops=0)
    if kind == "fc":
        w, b = _widths(case), case["batch"]
        e = 2 if case["dtype"] == "bf16" else 4
        weights = sum(x * y for x, y in zip(w, w[1:]))
        if case["mode"] == "forward":
            return dict(bytes=e * (weights + b * (w[0] + w[-1])), flops=2 * b * weights)
        return dict(bytes=e * (2 * weights + 2 * b * (w[0] + w[-1])), flops=6 * b * weights)
    R = case.get("R", 3)
    pad = case.get("pad", 1)
    px_in = case["N"] * case["H"] * case["W"]
    px_out = case["N"] * (case["H"] + 2 * pad - R + 1) * (case["W"] + 2 * pad - R + 1)
    filt = case["K"] * case["C"] * R * R
    flops = 6 * px_out * filt
    if kind == "conv":
        return dict(bytes=2 * (2 * px_in * case["C"] + 2 * px_out * case["K"] + 2 * filt), flops=flops)
    dims = [case["K"] * case["H"] * case["W"]] + _widths(case)
    weights = sum(x * y for x, y in zip(dims, dims[1:]))
    return dict(bytes=2 * (2 * px_in * case["C"] + 2 * filt + 2 * weights + 2 * case["N"] * dims[-1]),
                flops=flops + 6 * case["N"] * weights)


def tolerance(case):
    """Conversions move bytes.  Elsewhere sums may be taken in another order; what that changes is the rounding of stored
    bf16 results and, behind a ReLU, which side of zero a stored activation falls on.  About four times the largest
    difference seen between runs of one workload that cut its sums differently (no cuts, one to four cuts, other forms):
    f32 4e-7 to 1e-6; bf16 forward only 2e-4 (1.5e-3 through 8192-wide layers); bf16 steps 2.5e-3 with up to three
    layers, 1.2e-2 with four."""
    if case["kind"] == "retile":
        return "exact"
    if case["kind"] == "fc" and case["dtype"] == "f32":
        return dict(rel=4e-6)
    if case["kind"] == "conv":
        return dict(rel=1e-3)
    if case["kind"] == "fc" and case["mode"] == "forward":
        return dict(rel=4e-3)
    return dict(rel=1e-2 if len(_widths(case)) <= 4 else 4e-2)


# -------------------------------------------------------------------------------------------- the same in 64 bits

def _whole64(full, t, elem):
    """the shards of tiling t of a float64 matrix, one after the other at the 256-byte boundaries of `elem`-byte values"""
    rows, cols, unit = full.shape[0] >> t.count("R"), full.shape[1] >> t.count("C"), 256 // elem
    pitch = -(-rows * cols // unit) * unit
    whole = torch.zeros((1 << len(t)) * pitch, dtype=torch.float64, device=full.device)
    for s in range(1 << len(t)):
        rb, cb = _block_of(t, s)
        whole[s * pitch:s * pitch + rows * cols].view(rows, cols).copy_(full[rb * rows:(rb + 1) * rows, cb * cols:(cb + 1) * cols])
    return whole


def _full64(make, rows, cols, std, dtype):
    """the tensor `make.normal` cuts shards from, uncut"""
    return make.normal(rows, cols, "", std, dtype)[0].double()


def _fc64(x0, Ws, relus):
    """activations x[0..L] of a chain of fully-connected layers"""
    x = [x0]
    for W, relu in zip(Ws, relus):
        z = x[-1] @ W
        x.append(z.clamp_(min=0) if relu else z)
    return x


def _fc64_backward(x, Ws, relus, g):
    """weight gradients, and the gradient of x[0]"""
    dW = [None] * len(Ws)
    for l in reversed(range(len(Ws))):
        if relus[l]:
            g = g * (x[l + 1] > 0)
        dW[l] = x[l].t() @ g
        g = g @ Ws[l].t()
    return dW, g


def _windows(n, taps, pad, out):
    """per tap: (first input, first output, length) along one image dimension"""
    for r in range(taps):
        lo, hi = max(0, pad - r), min(out, n + pad - r)
        if hi > lo:
            yield r, lo + r - pad, lo, hi - lo


def _conv64(X, W, R, pad):
    """X: N,H,W,C; W: K,R,R,C -> N,P,Q,K"""
    n, h, w, _ = X.shape
    p, q = h + 2 * pad - R + 1, w + 2 * pad - R + 1
    Y = torch.zeros((n, p, q, W.shape[0]), dtype=torch.float64, device=X.device)
    for r, i, o, m in _windows(h, R, pad, p):
        for s, j, u, v in _windows(w, R, pad, q):
            Y[:, o:o + m, u:u + v] += (X[:, i:i + m, j:j + v].reshape(n * m * v, -1) @ W[:, r, s].t()).view(n, m, v, -1)
    return Y


def _conv64_backward(X, W, G, R, pad):
    """gradients of X and of W from that of the result"""
    n, h, w, c = X.shape
    p, q = G.shape[1:3]
    dX, dW = torch.zeros_like(X), torch.zeros_like(W)
    for r, i, o, m in _windows(h, R, pad, p):
        for s, j, u, v in _windows(w, R, pad, q):
            x = X[:, i:i + m, j:j + v].reshape(n * m * v, c)
            g = G[:, o:o + m, u:u + v].reshape(n * m * v, -1)
            dX[:, i:i + m, j:j + v] += (g @ W[:, r, s].contiguous()).view(n, m, v, c)
            dW[:, r, s] = g.t() @ x
    return dX, dW


def exact(case, seed):
    """What `run` returns on the same inputs, computed in 64 bits throughout (no stored value rounded in between).
    A conversion has no such value: its bytes are compared."""
    make = _Maker(seed)
    if case["kind"] == "retile":
        return None
    if case["kind"] == "fc":
        w, dt = _widths(case), _torch_dtype(case["dtype"])
        L, elem = len(w) - 1, 4 if case["dtype"] == "f32" else 2
        tx, tg, tw, _ = _fc_plan(tuple(w), case["batch"], case["k"], case["tiling"])
        x0 = _full64(make, case["batch"], w[0], 1.0, dt)
        Ws = [_full64(make, w[l], w[l + 1], case["w_std"], dt) for l in range(L)]
        relus = [l + 1 < L for l in range(L)]
        x = _fc64(x0, Ws, relus)
        if case["mode"] == "forward":
            return dict(x=[_whole64(x[l], tx[l], elem) for l in range(1, L + 1)])
        dW, g0 = _fc64_backward(x, Ws, relus, _full64(make, case["batch"], w[L], 1.0, dt))
        return dict(y=_whole64(x[L], tx[L], elem), dW=[_whole64(d, t, elem) for d, t in zip(dW, tw)],
                    dX=_whole64(g0, tg[0], elem))
    N, C, K, H, W = (case[n] for n in ("N", "C", "K", "H", "W"))
    R, pad, bf = case.get("R", 3), case.get("pad", 1), torch.bfloat16
    P, Q = H + 2 * pad - R + 1, W + 2 * pad - R + 1
    if case["kind"] == "conv":
        tX, tW, tY, tdY, tdX = _conv_plan(case)[0]
        X = _full64(make, N * H * W, C, 1.0, bf).view(N, H, W, C)
        F = _full64(make, K * R * R, C, 0.02, bf).view(K, R, R, C)
        G = _full64(make, N * P * Q, K, 1.0, bf).view(N, P, Q, K)
        dX, dF = _conv64_backward(X, F, G, R, pad)
        return dict(y=_whole64(_conv64(X, F, R, pad).view(-1, K), tY, 2), dW=_whole64(dF.view(-1, C), _swap(tW), 2),
                    dX=_whole64(dX.view(-1, C), tdX, 2))
    dims = [K * H * W] + _widths(case)
    n = len(dims) - 1
    p = _net_plan(case)[2]
    tx, tg, tw = p.x(), p.g(), p.w()
    X = _full64(make, N * H * W, C, 1.0, bf).view(N, H, W, C)
    F = _full64(make, K * 9, C, 1.5 / math.sqrt(9 * C), bf).view(K, 3, 3, C)
    Ws = [_full64(make, dims[i], dims[i + 1], 1.5 / math.sqrt(dims[i]), bf) for i in range(n)]
    relus = [i + 1 < n for i in range(n)]
    y1 = _conv64(X, F, 3, 1).clamp_(min=0)
    x = _fc64(y1.permute(0, 3, 1, 2).reshape(N, -1), Ws, relus)
    dW, g0 = _fc64_backward(x, Ws, relus, _full64(make, N, dims[n], 1.0, bf))
    dX, dF = _conv64_backward(X, F, g0.view(N, K, H, W).permute(0, 2, 3, 1) * (y1 > 0), 3, 1)
    return dict(y=_whole64(x[n], tx[n + 1], 2), dWf=[_whole64(d, t, 2) for d, t in zip(dW, tw[1:])],
                dWc=_whole64(dF.view(-1, C), _swap(tw[0]), 2), dX=_whole64(dX.view(-1, C), tg[0], 2))
