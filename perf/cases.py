"""The work that a user of this framework has it do, as cases that can be timed and compared.

A pass is what a streaming program does between two frames of its model: hand the frame's Q, K, V to
`global_attn`, its FFN-residual rows to `score_select`, and close the frame with `compact` -- for one
layer, for a stack of layers in one call, or layer by layer -- on a cache that is already full, which
is the state in which a bounded-cache stream spends its life.  Two kinds are different: `clip` starts
a new stream on an empty cache and feeds its first frames, and `checkpoint` writes a layer out to host
memory, reads it back into another handle and resumes there.

Values follow `synth`: Q, K, V are unit Gaussians, residual rows a Gaussian direction times a
log-normal norm (or a Pareto norm with repeated rows), frame 0 and the special tokens of the frames
that fill the cache are protected.  Residuals come from a long buffer that the passes walk along; when
its end is reached the walk starts again a few elements further on, so that a stream of thousands of
passes goes on seeing new scores instead of the same few frames.
"""
import math

import numpy as np
import torch

from paper_2603_05959_amd import binding as B
from paper_2603_05959_amd import synth

HEAD_DIM = 64
SPECIAL = 5                       # camera and register tokens at the head of a frame
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, M, budget, *, kind="stream", layers=1, per_layer=False, H=16, C=1024, dtype="bf16", out="f32",
          hybrid=False, smooth=False, resid="lognormal", static_ws=False, frames=1):
    case = {"kind": kind, "M": M, "B": budget, "layers": layers, "per_layer": per_layer, "H": H, "C": C, "dtype": dtype,
            "out": out, "hybrid": hybrid, "smooth": smooth, "resid": resid, "static_ws": static_ws, "frames": frames}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the camera head's cache: one token per frame, a budget of the frames that the aggregator holds;
        # nothing but latency and launches
        _case("camera-head", 1, 188),
        # the small all-fp32 stream with which the path is checked
        _case("tiny-f32", 65, 256, H=2, C=128, dtype="f32"),
        # a 518x392 layer with a short cache, by the entry point for programs that cannot allocate
        _case("layer-4k", 1041, 4096, static_ws=True),
        # a 518x392 layer as the paper runs it: hybrid scoring, smoothing, about 8 K tokens, outputs in the model's type
        _case("layer-8k-hybrid", 1041, 8192, out="bf16", hybrid=True, smooth=True),
        # the VGGT-sized layer of the benchmark's default line
        _case("layer-16k", 1374, 16384),
        # the long stream: heavy-tailed scores with exact ties, twice the cache
        _case("layer-32k-ties", 1374, 32768, resid="pareto"),
        # the largest budget of the 518x392 sweep
        _case("layer-64k", 1041, 65536, out="bf16"),
        # all 24 global-attention layers in one call per step (batched layers)
        _case("stack-16k", 1374, 16384, layers=24),
        # all 24 layers as a model's forward pass meets them, one after the other, in the paper's setting
        _case("stack-8k-by-layer", 1041, 8192, layers=24, per_layer=True, out="bf16", hybrid=True, smooth=True),
        # a new clip on kept buffers: handle, empty cache, the first ten frames (the ninth is the first to evict)
        _case("clip-start-8k", 1041, 8192, kind="clip", out="bf16", frames=10),
        # a 518x392 layer in fp32 throughout, as one compares a bf16 run with
        _case("layer-4k-f32", 1041, 4096, dtype="f32"),
        # a stream suspended and resumed: a layer exported to host memory, imported elsewhere, one more frame there
        _case("checkpoint-4k", 1041, 4096, kind="checkpoint", hybrid=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any frame size from one token to the VGGT frame, caches of a few to a few dozen
    frames, one layer or several, every option."""
    kind = rng.choice(["stream"] * 7 + ["stack"] * 4 + ["f32"] * 2 + ["clip"] * 2 + ["checkpoint"])
    H = rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 16, 16])
    C = rng.choice([H * HEAD_DIM, 128, 384, 1000, 1024])
    M = _log(rng, 1, 1374) if rng.random() < 0.6 else rng.randint(200, 1374)
    ratio = math.exp(rng.uniform(math.log(2.0), math.log(64.0)))
    smooth = M > 2 * SPECIAL and rng.random() < 0.3
    common = {"H": H, "C": C, "smooth": smooth, "resid": rng.choice(["lognormal", "lognormal", "pareto"])}
    if kind == "f32":
        return _case(None, M, min(4096, int(M * min(ratio, 16.0)) + rng.randint(0, 63)), dtype="f32", **common)
    # hybrid scoring reads the half-precision cache and takes up to 64 heads
    common.update(hybrid=rng.random() < 0.35, out=rng.choice(["f32", "bf16"]))
    budget = min(65536, int(M * ratio) + rng.randint(0, 127))
    if kind == "stack":
        budget = min(budget, 16384)
        layers = rng.choice([2, 3, 4, 6, 12, 24])
        while layers > 2 and layers * M * (budget + M) * H > 24 * 1374 * 17758 * 16:
            layers -= 1
        return _case(None, M, budget, layers=layers, per_layer=rng.random() < 0.5, **common)
    if kind == "clip":
        return _case(None, M, min(budget, 16384), kind="clip", frames=rng.randint(3, 12), **common)
    if kind == "checkpoint":
        return _case(None, min(M, 1041), max(min(budget, 4096), min(M, 1041)), kind="checkpoint", **common)
    return _case(None, M, budget, static_ws=rng.random() < 0.25, **common)


class Inputs:
    """A stream's frames on the GPU: a few distinct Q/K/V frames and a long walk of residual rows."""

    def __init__(self, case, seed):
        L, M, H, C = case["layers"], case["M"], case["H"], case["C"]
        dt = TYPES[case["dtype"]]
        gen = torch.Generator("cuda").manual_seed(seed)
        n_qkv = 3
        self.qkv = [tuple(torch.randn((L, M, H, HEAD_DIM), generator=gen, device="cuda", dtype=torch.float32).to(dt)
                          for _ in range(3)) for _ in range(n_qkv)]
        # residual rows: n_buf frames in memory, then the same memory again 8 elements (16 bytes or more) further on
        frame = L * M * C
        n_buf = max(4, min(4096, (64 << 20) // frame))
        pad_rows = -(-8 * 256 // C)
        rows = torch.randn((n_buf * L * M + pad_rows, C), generator=gen, device="cuda", dtype=torch.float32)
        z = torch.randn((rows.shape[0], 1), generator=gen, device="cuda", dtype=torch.float32)
        if case["resid"] == "pareto":
            u = torch.rand((rows.shape[0], 1), generator=gen, device="cuda", dtype=torch.float32)
            norm = (1.0 - u).clamp_min(1e-7) ** (-1.0 / 1.5)
        else:
            norm = torch.exp(z)
        rows = rows * (norm / math.sqrt(C))
        if case["resid"] == "pareto":               # one row in twenty repeats another one exactly
            n_dup = rows.shape[0] // 20
            dst = torch.randperm(rows.shape[0], generator=gen, device="cuda")[:n_dup]
            src = torch.randint(0, rows.shape[0], (n_dup,), generator=gen, device="cuda")
            rows[dst] = rows[src].clone()
        self.flat = rows.to(dt).reshape(-1)
        n_win = min(4096, n_buf * 256)
        # 16 bytes at a time in the walk; every window is a view [L, M, C]
        self.windows = [self.flat[w % n_buf * frame + w // n_buf * 8:][:frame].view(L, M, C) for w in range(n_win)]
        if case["per_layer"]:
            self.qkv = [tuple([x[l] for l in range(L)] for x in f) for f in self.qkv]
            self.windows = [[w[l] for l in range(L)] for w in self.windows[:512]]
        self.t = 0

    def next(self):
        t = self.t
        self.t = t + 1
        return self.qkv[t % len(self.qkv)], self.windows[t % len(self.windows)]


def _smoothing(case):
    """(alpha, rows, columns, special tokens, 3x3 kernel) of Eq. 6, or None."""
    if not case["smooth"]:
        return None
    grid = synth.StreamConfig("", case["M"], case["H"], HEAD_DIM, case["C"], case["B"], 1, 1, case["dtype"], SPECIAL, "", "")
    ph, pw = synth.patch_grid(grid)
    return 0.5, ph, pw, SPECIAL, synth.gaussian_kernel3(1.0)


def _make_cache(case):
    return B.Cache(case["layers"], case["H"], HEAD_DIM, case["M"], case["C"], case["B"], case["dtype"], out_dtype=case["out"],
                   smooth=_smoothing(case), hybrid_beta=0.5 if case["hybrid"] else None)


def _anchors(case, t):
    """Frame 0, then the special tokens of the frames that fill the cache, up to a tenth of the budget
    beyond frame 0 (and never more than the budget holds beside a frame)."""
    M, budget = case["M"], case["B"]
    a = np.zeros(M, np.uint8)
    if t == 0:
        a[: min(M, budget // 2)] = 1
    elif t * SPECIAL <= budget // 10 and M > SPECIAL:
        a[:SPECIAL] = 1
    return torch.from_numpy(np.repeat(a[None], case["layers"], axis=0)).cuda()


class State:
    def __init__(self, case, seed):
        self.case = case
        self.inputs = Inputs(case, seed)
        self.cache = _make_cache(case)
        self.out = self.cache.new_output()
        self.outs = [self.out[l] for l in range(case["layers"])]
        if case["kind"] == "clip":
            self.anchors = [_anchors(case, t) for t in range(case["frames"])]
            self.clip_outs = [self.cache.new_output() for _ in range(case["frames"])]
            return
        for t in range(-(-case["B"] // case["M"]) + 1):      # until the cache is full and has evicted once
            self.step(_anchors(case, t))
        if case["kind"] == "checkpoint":
            n, row = case["B"], (case["H"], HEAD_DIM)
            store = np.uint16 if case["dtype"] == "bf16" else np.float32
            self.host = (np.zeros(n, np.uint32), np.zeros((n, *row), store), np.zeros((n, *row), store),
                         np.zeros(n, np.float32), np.zeros(n, np.uint8))
            self.resumed = _make_cache(case)

    def step(self, anchors=None):
        (q, k, v), r = self.inputs.next()
        c, case = self.cache, self.case
        if case["per_layer"]:
            for l in range(case["layers"]):
                c.step(q[l], k[l], v[l], r[l], None if anchors is None else anchors[l], self.outs[l], layer=l)
        elif case["static_ws"]:
            B.ovggt_global_attn_static_ws(c.h, 0, q, k, v, self.out, c.stream)
            c.score_select(r, anchors, 0)
            c.compact(0)
        else:
            c.step(q, k, v, r, anchors, self.out)
        return self.out


def prepare(case, seed):
    return State(case, seed)


def _run_clip(s):
    """A new stream on the buffers of the last one: a handle of its own, then its first frames."""
    c = s.cache
    h = B.ovggt_cache_init(c.cfg, c.bufs.kv, c.bufs.meta, c.bufs.ws, c.stream)
    for a, out in zip(s.anchors, s.clip_outs):
        (q, k, v), r = s.inputs.next()
        B.ovggt_global_attn(h, B.OVGGT_ALL_LAYERS, q, k, v, out, c.stream)
        B.ovggt_score_select(h, B.OVGGT_ALL_LAYERS, r, a, c.stream)
        B.ovggt_cache_compact(h, B.OVGGT_ALL_LAYERS, c.stream)
    B.ovggt_cache_destroy(h)
    return s.clip_outs


def _run_checkpoint(s):
    """Layer 0 to host memory, from there into another handle, and the stream's next frame on that one."""
    c, to = s.cache, s.resumed
    ids, k, v, ss, flags = s.host
    B.ovggt_cache_export(c.h, 0, ids, k, v, ss, flags, c.stream)
    B.ovggt_cache_import(to.h, 0, len(ids), c.frames(0), ids, k, v, ss, flags, to.stream)
    (q, kn, vn), r = s.inputs.next()
    to.step(q, kn, vn, r, None, s.out, 0)
    return [s.out, *s.host]


def run(s):
    if s.case["kind"] == "clip":
        return _run_clip(s)
    if s.case["kind"] == "checkpoint":
        return _run_checkpoint(s)
    return s.step()


def _step_work(case, n_old):
    """One frame of one layer on n_old cached tokens: K and V of the cache are read once, the frame's
    Q, K, V and residual rows are read, its K and V join the cache, O is written, and every score and
    flag is looked at."""
    M, H, C = case["M"], case["H"], case["C"]
    e = 2 if case["dtype"] == "bf16" else 4
    row = H * HEAD_DIM
    n = n_old + M
    byts = 2 * n_old * row * e + 3 * M * row * e + 2 * M * row * e + M * row * (4 if case["out"] == "f32" else 2)
    byts += M * C * e + 5 * n
    flops = 4.0 * M * n * row + 2.0 * M * C
    if case["hybrid"] and n > case["B"]:
        flops += 4.0 * n_old * row                  # each old key against the centroid, and its own length
    return byts, flops


def work(case):
    if case["kind"] == "clip":
        sizes = [min(t * case["M"], case["B"]) for t in range(case["frames"])]
    else:
        sizes = [case["B"]]
    parts = [_step_work(case, n) for n in sizes]
    byts, flops = sum(p[0] for p in parts) * case["layers"], sum(p[1] for p in parts) * case["layers"]
    if case["kind"] == "checkpoint":                # read and written on each side of the bus, both ways
        e = 2 if case["dtype"] == "bf16" else 4
        byts += 4 * case["B"] * (2 * case["H"] * HEAD_DIM * e + 9)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Attention outputs, about four times what they were seen to be off from the same sums in 64 bits
    (rel 3e-4 and max 2.4e-3 with half-precision weights, 1.7e-3 and 5e-3 rounded to bf16 on top, 7e-7
    and 7e-6 in fp32); ids, flags and exported K and V are whole numbers and stay the same."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 1.2e-3, "max": 1e-2}


# ---- the same passes in plain torch: attention in 64 bits, on the tokens that Eq. 8 keeps ------------
# Which tokens those are hangs on the last bit of a score, so scores follow the sequence that defines
# them: single fp32 operations, sums as balanced trees over neighbours.

def _tree(x):
    """Row sums of [n, w] as a balanced binary tree over neighbours, zero-padded to a power of two."""
    x = torch.nn.functional.pad(x, (0, (1 << (x.shape[1] - 1).bit_length()) - x.shape[1]))
    while x.shape[1] > 1:
        x = x[:, 0::2] + x[:, 1::2]
    return x[:, 0]


def _sqrt(x):
    return x.double().sqrt().float()                # correctly rounded


def _div(x, y):
    return (x.double() / y.double()).float()        # correctly rounded


def _min_max(x, weight):
    lo, hi = x.min(), x.max()
    unit = torch.zeros_like(x) if bool(lo == hi) else _div(x - lo, hi - lo)
    return weight * unit


class ExactLayer:
    """One layer's cache in the order of arrival: keys, values, rank keys and protection of the resident tokens."""

    def __init__(self, case):
        self.case, self.smooth = case, _smoothing(case)
        self.k = self.v = torch.zeros((0, case["H"], HEAD_DIM), dtype=TYPES[case["dtype"]], device="cuda")
        self.key = torch.zeros(0, device="cuda")
        self.kept = torch.zeros(0, dtype=torch.bool, device="cuda")

    def append(self, k, v):
        self.k, self.v = torch.cat([self.k, k]), torch.cat([self.v, v])

    def attend(self, q):
        out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        for h in range(q.shape[1]):
            s = torch.mm(q[:, h].double(), self.k[:, h].double().t().contiguous()) / math.sqrt(HEAD_DIM)
            out[:, h] = torch.mm(torch.softmax(s, dim=1), self.v[:, h].double())
        return out

    def close(self, r, anchors):
        """Scores of the frame just appended, then the budget."""
        r = r.float()
        key = _tree(r * r)
        if self.smooth is not None:
            alpha, ph, pw, first, g = self.smooth
            key = _sqrt(key)
            grid = torch.nn.functional.pad(key[first:].view(1, 1, ph, pw), (1, 1, 1, 1), mode="replicate")[0, 0]
            conv = None
            for t in range(9):
                prod = float(g[t // 3, t % 3]) * grid[t // 3:t // 3 + ph, t % 3:t % 3 + pw]
                conv = prod if conv is None else conv + prod
            key[first:] = alpha * conv.reshape(-1) + (1.0 - alpha) * key[first:]
        n_old = len(self.key)
        self.key = torch.cat([self.key, key])
        new = torch.zeros(len(key), dtype=torch.bool, device="cuda") if anchors is None else anchors.bool()
        self.kept = torch.cat([self.kept, new])
        budget = self.case["B"]
        if len(self.key) <= budget:
            return
        free = torch.nonzero(~self.kept)[:, 0]
        if self.case["hybrid"]:
            self._rank_by_diversity(free[free < n_old], free[free >= n_old])
        best = torch.sort(self.key[free], descending=True, stable=True).indices[:budget - int(self.kept.sum())]
        stay = torch.sort(torch.cat([torch.nonzero(self.kept)[:, 0], free[best]])).values
        self.k, self.v, self.key, self.kept = self.k[stay], self.v[stay], self.key[stay], self.kept[stay]

    def _rank_by_diversity(self, hist, new):
        """Eq. 7: min-max of 1 - cos(key, centroid) for the history, of the scores for the new frame."""
        if len(hist):
            k = self.k[hist].half().float().reshape(len(hist), -1)
            total = torch.zeros(k.shape[1], dtype=torch.int64, device="cuda")
            for part in k.split(4096):
                total += (part.double() * 2.0 ** 24).long().sum(0)
            c = (total.double().float() * 2.0 ** -24)[None]
            den = _sqrt(_tree(k * k)) * _sqrt(_tree(c * c))
            cos = torch.where(den == 0, 0.0, _div(_tree(k * c), den))
            self.key[hist] = _min_max(1.0 - cos, 0.5)
        if len(new):
            s = self.key[new]
            self.key[new] = _min_max(s if self.smooth is not None else _sqrt(s), 0.5)


def exact(case, seed):
    """The first pass on these inputs; ids, flags, scores and the exported rows are compared as they are."""
    inputs = Inputs(case, seed)
    layers = [ExactLayer(case) for _ in range(case["layers"])]

    def frame(anchors, attend, close=True):
        (q, k, v), r = inputs.next()
        outs = []
        for l, x in enumerate(layers):
            x.append(k[l], v[l])
            if attend:
                outs.append(x.attend(q[l]))
            if close:
                x.close(r[l], None if anchors is None else anchors[l])
        return torch.stack(outs) if attend else None

    if case["kind"] == "clip":
        return [frame(_anchors(case, t), True) for t in range(case["frames"])]
    for t in range(-(-case["B"] // case["M"]) + 1):
        frame(_anchors(case, t), False)
    out = frame(None, True, close=False)
    return [out, None, None, None, None, None] if case["kind"] == "checkpoint" else out
