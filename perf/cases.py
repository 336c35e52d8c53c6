"""Performance cases of the mask-aware denoising step.

What a program that serves editing requests runs, through the library's public
calls: one transformer block over the packed masked rows (``gather_rows`` +
``block_forward``, the unit every denoising step repeats per layer), the
recomputation of the unmasked tokens' K/V from cached block inputs
(``recompute_kv``, the Y-caching variant) and whole denoising steps
(``stack_forward``) with the K/V cache resident in HBM or streamed from pinned
host memory. A case is a dict of sizes; every request's mask has a fixed number
of masked tokens (its ratio times the grid), at places drawn from the seed.

``exact`` is the same computation in plain torch float64, without rounding
between the operations.
"""
import math

import numpy as np
import torch

from paper_2505_20600_amd import maskstep as MS
from paper_2505_20600_amd import workloads as W

DEV = "cuda:0"


def _case(name, op, d, heads, grid_h, grid_w, batch, lo, hi, layers=1, text=0, dual=False, mlp=4, dtype="bf16",
          prefix=0):
    """lo, hi: mask ratios of the first and the last request, the others spread evenly over their logarithm."""
    return {"name": name, "op": op, "layers": layers, "d": d, "heads": heads, "mlp": mlp, "grid_h": grid_h,
            "grid_w": grid_w, "text": text, "dual": dual, "batch": batch, "lo": lo, "hi": hi, "dtype": dtype,
            "prefix": prefix}


def listed():
    return [
        # a float32 model's block on a 32 x 32 latent, a fifth of it edited: the smallest call, bound by launches
        _case("block_d256_fp32", "block", 256, 4, 32, 32, 1, 0.2, 0.2, dtype="fp32"),
        # interactive edit of a small region: one request, few rows, weights and cached K/V read for little work
        _case("block_d768_r05", "block", 768, 12, 64, 64, 1, 0.05, 0.05),
        # the same model at the upper end of the usual mask ratios
        _case("block_d768_r35", "block", 768, 12, 64, 64, 1, 0.35, 0.35),
        # many small latents batched together (thumbnails, previews)
        _case("block_d512_batch16", "block", 512, 8, 32, 32, 16, 0.05, 0.5),
        # one request of the mid-sized model (head_dim 72)
        _case("block_d1152_r25", "block", 1152, 16, 64, 64, 1, 0.25, 0.25),
        # a full serving batch of that model, mask ratios as in production traces
        _case("block_d1152_batch8", "block", 1152, 16, 64, 64, 8, 0.03, 0.8),
        # every token masked: the template's own pass that fills the cache, or an edit of the whole image
        _case("block_d1152_all", "block", 1152, 16, 64, 64, 1, 1.0, 1.0),
        # another head width, a portrait-format latent with odd sides, three requests
        _case("block_d1152_hd96_ragged", "block", 1152, 12, 61, 45, 3, 0.1, 0.6),
        # a large two-stream model's block: 512 text rows per request always recomputed, four requests
        _case("block_d3072_text_batch4", "block", 3072, 24, 64, 64, 4, 0.1, 0.4, text=512, dual=True),
        # Y caching: K/V of the unmasked tokens from the cached block inputs, the same model and batch
        _case("recompute_d3072_batch4", "recompute", 3072, 24, 64, 64, 4, 0.1, 0.4, text=512, dual=True),
        # a whole denoising step, K/V cache resident in HBM
        _case("step_d768_12layers", "step", 768, 12, 64, 64, 1, 0.3, 0.3, layers=12),
        # a whole denoising step, K/V cache streamed from pinned host memory, first two blocks over every token
        _case("step_d1152_streamed", "streamed", 1152, 16, 64, 64, 1, 0.25, 0.25, layers=28, prefix=2),
    ]


# head widths a draw takes, the common ones more often
_HEAD_DIMS = (64, 64, 64, 72, 72, 128, 128, 128, 32, 40, 48, 80, 88, 96, 104, 112, 120)


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    most = 0.9 * max(work(c)["flops"] for c in listed() if c["op"] == "block")
    while True:
        op = rng.choice(("block", "block", "block", "block", "recompute", "step", "streamed"))
        dtype = "fp32" if rng.random() < 0.1 else "bf16"
        hd = rng.choice((32, 40, 64)) if dtype == "fp32" else rng.choice(_HEAD_DIMS)
        unit = hd * 64 // math.gcd(hd, 64)
        target = _log_uniform(rng, 256, 1024 if dtype == "fp32" else 3072)
        d = max(1, round(target / unit)) * unit
        if d > (1024 if dtype == "fp32" else 3072):
            continue
        batch = int(_log_uniform(rng, 1, 9))
        lo = _log_uniform(rng, 0.03, 0.6)
        hi = lo if batch == 1 else min(1.0, lo * _log_uniform(rng, 1.0, 8.0))
        text = rng.choice((0, 0, 0, rng.randint(1, 512)))
        c = {"op": op, "layers": 1, "d": d, "heads": d // hd, "mlp": rng.choice((4, 4, 4, 2, 3)),
             "grid_h": int(_log_uniform(rng, 16, 73)), "grid_w": int(_log_uniform(rng, 16, 73)), "text": text,
             "dual": text > 0 and rng.random() < 0.5, "batch": batch, "lo": lo, "hi": hi, "dtype": dtype, "prefix": 0}
        if op in ("step", "streamed"):
            c["layers"] = rng.randint(2, 12)
            c["prefix"] = rng.randint(0, 2) if op == "streamed" else 0
        w = work(c)
        if w["flops"] > most or w["bytes"] > 1.5e9:
            continue
        return c


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------


def _shape(case):
    return W.ModelShape("case", case["layers"], case["d"], case["heads"], case["mlp"], case["grid_h"], case["grid_w"],
                        n_text=case["text"], dual_stream=case["dual"], dtype=case["dtype"], batch=case["batch"])


def _masked_counts(case):
    """Masked image tokens of each request."""
    n, B = case["grid_h"] * case["grid_w"], case["batch"]
    out = []
    for b in range(B):
        r = case["lo"] * (case["hi"] / case["lo"]) ** (b / (B - 1) if B > 1 else 0.0)
        out.append(min(n, max(1, round(r * n))))
    return out


def work(case):
    """Each block's weights, the cached K/V of the unmasked tokens (or the block inputs they are recomputed from) and
    the packed rows read once, the fresh K/V rows and the output rows written once."""
    d, f, B = case["d"], case["mlp"] * case["d"], case["batch"]
    N = case["grid_h"] * case["grid_w"]
    T = N + case["text"]
    e = 2 if case["dtype"] == "bf16" else 4
    counts = _masked_counts(case)
    U = sum(N - c for c in counts)
    if case["op"] == "recompute":
        return {"bytes": e * (2 * d * d + U * d + 2 * U * d), "flops": 4 * U * d * d}
    rows = [c + case["text"] for c in counts]
    M = sum(rows)
    sets = 2 if case["dual"] else 1
    flops = bytes_ = 0
    for l in range(case["layers"]):
        dense = l < case["prefix"]
        # the last block of a dense prefix needs the unmasked tokens for their K/V only
        inner = dense and l < case["prefix"] - 1
        R, att = (B * T, B * T * T) if inner else (M, sum(r * T for r in rows))
        kvrows = B * T if dense else M
        flops += 4 * kvrows * d * d + 2 * R * d * d * (2 + 2 * case["mlp"]) + 4 * att * d
        bytes_ += e * sets * (4 * d * d + 2 * d * f) + e * 2 * d * (B * T)
        if not dense:
            bytes_ += e * 2 * d * M      # the masked rows' fresh K/V, written over the cached ones
    if case["op"] == "block":
        bytes_ += e * 2 * M * d
    else:
        bytes_ += e * (M * d + B * T * d)   # the rows read, the whole output written ...
        bytes_ += e * (B * T - M) * d       # ... from the cached output where nothing is recomputed
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times the distance of the library's outputs to ``exact``: in bf16 the activations, the attention
    weights and the outputs are rounded (2^-9 each) and a block leaves 2.4e-3 to 3.1e-3 of it in its outputs; a stack
    adds its blocks' errors (1.1e-2 after 28). float32: up to 2.1e-7 after one block."""
    if case["dtype"] == "fp32":
        return {"rel": 2e-6 if case["layers"] == 1 else 5e-6, "max": 1e-4}
    if case["op"] in ("step", "streamed"):
        return {"rel": 2.5e-2, "max": 0.5}
    return {"rel": 1e-2, "max": 0.2}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _masks(case, seed):
    """uint8 [B][N]: the union of one to four ellipses per request, cut to the request's number of tokens."""
    h, w = case["grid_h"], case["grid_w"]
    g = np.random.default_rng([seed, 17])
    yy, xx = np.meshgrid(np.arange(h) + 0.5, np.arange(w) + 0.5, indexing="ij")
    out = np.zeros((case["batch"], h * w), np.uint8)
    for b, count in enumerate(_masked_counts(case)):
        score = np.full((h, w), np.inf)
        for _ in range(int(g.integers(1, 5))):
            cy, cx, aspect, size = g.uniform(0, h), g.uniform(0, w), g.uniform(0.5, 2.0), g.uniform(0.5, 1.5)
            t = g.uniform(0, math.pi)
            u = (xx - cx) * math.cos(t) + (yy - cy) * math.sin(t)
            v = (yy - cy) * math.cos(t) - (xx - cx) * math.sin(t)
            score = np.minimum(score, (u / (size * math.sqrt(aspect))) ** 2 + (v * math.sqrt(aspect) / size) ** 2)
        out[b, np.argsort(score.reshape(-1), kind="stable")[:count]] = 1
    return out


def _inputs(case, seed):
    """Weights (N(0, 0.02), LayerNorm near one), hidden states N(0, 1), caches of the spread that projections of
    normalised rows have; all on the GPU in the model's type."""
    tdt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device=DEV).manual_seed(seed)
    d, f, B, L = case["d"], case["mlp"] * case["d"], case["batch"], case["layers"]
    N = case["grid_h"] * case["grid_w"]
    T = N + case["text"]

    def rand(*shape, std=1.0, mean=0.0):
        return torch.randn(*shape, device=DEV, dtype=tdt, generator=g).mul_(std).add_(mean)

    def weights():
        return {"ln1_g": rand(d, std=0.1, mean=1.0), "ln1_b": rand(d, std=0.1),
                "w_qkv": rand(3 * d, d, std=0.02), "b_qkv": rand(3 * d, std=0.02),
                "w_o": rand(d, d, std=0.02), "b_o": rand(d, std=0.02),
                "ln2_g": rand(d, std=0.1, mean=1.0), "ln2_b": rand(d, std=0.1),
                "w_1": rand(f, d, std=0.02), "b_1": rand(f, std=0.02),
                "w_2": rand(d, f, std=0.02), "b_2": rand(d, std=0.02)}

    layers = [(weights(), weights()) if case["dual"] else weights() for _ in range(L)]
    kv_std = 0.02 * math.sqrt(d)
    x = rand(B, T, d)
    mask = torch.as_tensor(_masks(case, seed)).to(DEV)
    s = {"layers": layers, "x": x, "mask": mask}
    if case["op"] == "recompute":
        s["yin"] = rand(B, N, d)
        s["kv"] = [rand(B, T, 2, d, std=kv_std)]
    elif case["op"] == "streamed":
        s["kv_host"] = [rand(B, N, 2, d, std=kv_std) for _ in range(L)]   # prepare() takes them to pinned memory
    else:
        s["kv"] = [rand(B, T, 2, d, std=kv_std) for _ in range(L)]
    if case["op"] in ("step", "streamed"):
        s["yc"] = rand(B, T, d)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    shape = _shape(case)
    desc = MS.model_desc(shape)
    B = case["batch"]
    ws = torch.empty(MS.mask_workspace_bytes(desc, B), dtype=torch.uint8, device=DEV)
    step = MS.MaskStep(desc, B, s["mask"], ws)
    s.update(case=case, step=step)
    if case["op"] == "block":
        s["xm"] = torch.empty(step.info().rows, case["d"], device=DEV, dtype=s["x"].dtype)
    if case["op"] in ("step", "streamed"):
        s["wc"] = MS.weights_array(s["layers"])
        s["y"] = torch.empty_like(s["x"])
    if case["op"] == "streamed":
        T, d = case["text"] + case["grid_h"] * case["grid_w"], case["d"]
        host = []
        for t in s["kv_host"]:
            p = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
            p.copy_(t)
            host.append(p)
        s["kv_host"] = host
        s["slots"] = [torch.empty(B, T, 2, d, device=DEV, dtype=s["x"].dtype) for _ in range(case["layers"])]
        s["copy_stream"] = torch.cuda.Stream()
        step.set_dense_prefix(case["prefix"])
    return s


def run(state):
    case, step = state["case"], state["step"]
    if case["op"] == "block":
        step.gather_rows(state["x"], state["xm"])
        step.block_forward(0, state["layers"][0], state["xm"], state["kv"][0])
        return {"xm": state["xm"], "kv": state["kv"][0]}
    if case["op"] == "recompute":
        step.recompute_kv(0, state["layers"][0], state["yin"], state["kv"][0])
        return {"kv": state["kv"][0]}
    if case["op"] == "step":
        step.stack_forward(state["wc"], state["x"], state["yc"], state["kv"], state["y"])
        return {"y": state["y"], "kv": state["kv"]}
    step.stack_forward(state["wc"], state["x"], state["yc"], state["kv_host"], state["y"], pinned=True,
                       slots=state["slots"], copy_stream=state["copy_stream"], loads_ahead=True)
    return {"y": state["y"]}


# ---------------------------------------------------------------------------
# the same in float64
# ---------------------------------------------------------------------------


def _ln(x, g, b):
    m = x.mean(-1, keepdim=True)
    v = ((x - m) ** 2).mean(-1, keepdim=True)
    return (x - m) / torch.sqrt(v + 1e-5) * g + b


def _lin(x, w, b):
    return x @ w.t().contiguous() + b


def _rows_apply(fn, x, is_text, w):
    """fn(rows, weight set): text rows with the text set of a two-stream model."""
    if not isinstance(w, tuple):
        return fn(x, w)
    parts_i, parts_t = fn(x[~is_text], w[0]), fn(x[is_text], w[1])
    out = torch.empty((x.shape[0], parts_i.shape[1]), dtype=x.dtype, device=x.device)
    out[~is_text], out[is_text] = parts_i, parts_t
    return out


def _attend(q, kv, heads):
    """q [m][d] over kv [T][2][d]."""
    m, d = q.shape
    hd = d // heads
    o = torch.empty_like(q)
    for h in range(heads):
        c = slice(h * hd, (h + 1) * hd)
        k, v = kv[:, 0, c].contiguous(), kv[:, 1, c].contiguous()
        for r in range(0, m, 4096):
            p = torch.softmax(q[r:r + 4096, c].contiguous() @ k.t().contiguous() / math.sqrt(hd), dim=-1)
            o[r:r + 4096, c] = p @ v
    return o


def _exact_block(case, w, x, rows, kv):
    """x [T][d] of one request: its `rows` (sorted token indices) after the block; kv [T][2][d] gets their K/V."""
    d = case["d"]
    is_text = rows < case["text"]
    xm = x[rows]
    qkv = _rows_apply(lambda r, p: _lin(_ln(r, p["ln1_g"], p["ln1_b"]), p["w_qkv"], p["b_qkv"]), xm, is_text, w)
    kv[rows] = qkv[:, d:].reshape(-1, 2, d)
    o = _attend(qkv[:, :d].contiguous(), kv, case["heads"])
    h = xm + _rows_apply(lambda r, p: _lin(r, p["w_o"], p["b_o"]), o, is_text, w)
    return h + _rows_apply(
        lambda r, p: _lin(torch.nn.functional.gelu(_lin(_ln(r, p["ln2_g"], p["ln2_b"]), p["w_1"], p["b_1"])),
                          p["w_2"], p["b_2"]), h, is_text, w)


def exact(case, seed):
    s = _inputs(case, seed)
    B, d, text = case["batch"], case["d"], case["text"]
    T = text + case["grid_h"] * case["grid_w"]

    def up(w):
        return tuple(up(p) for p in w) if isinstance(w, tuple) else {k: v.double() for k, v in w.items()}

    mask = s["mask"] != 0
    full = torch.cat([torch.ones(B, text, dtype=torch.bool, device=DEV), mask], dim=1)
    rows = [full[b].nonzero().reshape(-1) for b in range(B)]
    if case["op"] == "recompute":
        w = up(s["layers"][0])
        w = w[0] if isinstance(w, tuple) else w
        kv = s["kv"][0].double()
        for b in range(B):
            if text == 0 and not bool(mask[b].any()):
                continue
            u = (~mask[b]).nonzero().reshape(-1)
            r = _lin(_ln(s["yin"][b][u].double(), w["ln1_g"], w["ln1_b"]), w["w_qkv"][d:], w["b_qkv"][d:])
            kv[b, text + u] = r.reshape(-1, 2, d)
        return {"kv": kv}
    xs = [s["x"][b].double() for b in range(B)]
    kvs = []
    for l in range(case["layers"]):
        w = up(s["layers"][l])
        if case["op"] == "streamed":
            kv = torch.zeros(B, T, 2, d, device=DEV, dtype=torch.float64)
            kv[:, text:] = s["kv_host"][l].double()
        else:
            kv = s["kv"][l].double()
        for b in range(B):
            r = torch.arange(T, device=DEV) if l < case["prefix"] else rows[b]
            out = _exact_block(case, w, xs[b], r, kv[b])
            xs[b] = xs[b].clone()
            xs[b][r] = out
        if case["op"] != "streamed":
            kvs.append(kv)
    if case["op"] == "block":
        if case["dual"]:   # text rows of all requests, then the image rows
            xm = torch.cat([xs[b][rows[b][:text]] for b in range(B)] + [xs[b][rows[b][text:]] for b in range(B)])
        else:
            xm = torch.cat([xs[b][rows[b]] for b in range(B)])
        return {"xm": xm, "kv": kvs[0]}
    y = s["yc"].double()
    for b in range(B):
        y[b, rows[b]] = xs[b][rows[b]]
    return {"y": y} if case["op"] == "streamed" else {"y": y, "kv": kvs}
