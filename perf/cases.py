"""The restoration work that performance is measured on, and the ranges it stands for.

A case names one path through the public entry points and the sizes it runs at; `prepare` makes
what a serving program holds before the call (a context with packed weights and a registered
paged pool, hidden states, positions, block tables, a chunk store), `run` makes the call.  Model
widths are those of this repository's workloads.  The values follow the same recipe: weights
N(0, 0.02^2), gains near 1, hidden states N(0, 1) with 1 % of the channels scaled by 20, pages a
random permutation of a pool 25 % larger than needed.
"""
import ctypes
import random

import numpy as np
import torch

import paper_2410_05004_amd as hc

BLOCK = 16                 # tokens per page
CHUNK = 256                # tokens per chunk of the host store

# width: (d_model, KV heads, head dim, RoPE theta, RoPE style, normalisation)
WIDTHS = {
    "d256": (256, 4, 64, 1e4, 0, "rms"),
    "d4096": (4096, 32, 128, 1e4, 0, "rms"),
    "d4096-gqa": (4096, 8, 128, 5e5, 0, "rms"),
    "d4096-gqa-bias": (4096, 8, 128, 5e5, 1, "rms+bias"),
    "d5120": (5120, 40, 128, 1e4, 0, "rms"),
    "d7168-layernorm": (7168, 56, 128, 1e4, 2, "layer"),
    "d8192-gqa": (8192, 8, 128, 5e5, 0, "rms"),
}


def listed():
    return [
        # one layer of the tiny model: nothing but launch and latency
        dict(name="layer-tiny", path="layer", width="d256", layers=1, tokens=128, offset=0),
        # one layer of a short turn of a grouped-query model, layers arriving one at a time
        dict(name="layer-turn", path="layer", width="d4096-gqa", layers=1, tokens=37, offset=0),
        # one layer of an ordinary conversation, interleaved rotation, K/V biases, odd length
        dict(name="layer-bias", path="layer", width="d4096-gqa-bias", layers=1, tokens=2501, offset=0),
        # one layer of a multi-head model, a length just past what fills the device evenly
        dict(name="layer-mha", path="layer", width="d5120", layers=1, tokens=1601, offset=0),
        # all layers of a short context whose hidden states were kept on the device
        dict(name="all-short", path="layers", width="d4096-gqa", layers=32, tokens=300, offset=0),
        # all layers of an 8K context: the workload the headline rate is quoted on
        dict(name="all-8k", path="layers", width="d4096-gqa", layers=32, tokens=8192, offset=0),
        # eight layers of a long context of the largest model, continuing inside a page
        dict(name="all-long", path="layers", width="d8192-gqa", layers=8, tokens=32768, offset=1000),
        # eight layers of a LayerNorm model with biases and no rotation
        dict(name="all-layernorm", path="layers", width="d7168-layernorm", layers=8, tokens=2048, offset=0),
        # one layer of a batch of requests restored together
        dict(name="batch", path="ragged", width="d5120", layers=1, tokens=34175, contexts=16),
        # all layers of a context streamed from the pinned host store, starting inside a chunk
        dict(name="from-store", path="store", width="d4096-gqa", layers=32, tokens=1000, offset=100),
        # KV offload of one layer: a context's rows read out of its pages, and put into other pages
        dict(name="offload", path="rows", width="d4096", layers=1, tokens=2048, offset=0),
        # saving a fused step: a prefill beside decoding contexts, through four layers
        dict(name="save-step", path="save", width="d4096-gqa", layers=4, tokens=1001, contexts=11),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    path = rng.choice(["layer"] * 5 + ["layers"] * 4 + ["ragged"] * 2 + ["store", "rows", "save"])
    width = rng.choice([w for w in WIDTHS if w != "d256" or path in ("layer", "layers")])
    d, heads, hd = WIDTHS[width][:3]
    d_kv = heads * hd
    if path == "layer":
        return dict(path=path, width=width, layers=1, tokens=_log_int(rng, 1, 16384), offset=rng.choice([0, 0, rng.randrange(4096)]))
    if path == "layers":
        layers = rng.choice([4, 8, 12, 16, 32])
        # no more work than the largest listed case, at most 4 GiB of hidden states
        most = min(32768, int(2 ** 43 / (4 * d * d_kv * layers)), 2 ** 31 // (d * layers))
        return dict(path=path, width=width, layers=layers, tokens=_log_int(rng, 16, most), offset=rng.choice([0, 0, rng.randrange(4096)]))
    if path == "ragged":
        n = _log_int(rng, 2, 64)
        return dict(path=path, width=width, layers=1, tokens=n * _log_int(rng, 8, 32768 // n) + rng.randrange(n), contexts=n)
    if path == "store":
        layers = rng.choice([8, 16, 32])
        most = 2 ** 28 // (2 * d * layers)          # at most 256 MiB over the host link
        return dict(path=path, width=width, layers=layers, tokens=_log_int(rng, 16, most), offset=rng.randrange(CHUNK))
    if path == "rows":
        return dict(path=path, width=width, layers=1, tokens=_log_int(rng, 1, 8192), offset=rng.choice([0, rng.randrange(1024)]))
    contexts = rng.randrange(1, 12)
    return dict(path=path, width=width, layers=rng.choice([1, 2, 4]), tokens=_log_int(rng, 1, 1024), contexts=contexts)


def lengths(case):
    """Token counts of the contexts of a batch: uneven, at least 1 each, adding up to `tokens`."""
    r = random.Random("%d-%d" % (case["tokens"], case["contexts"]))
    n, total = case["contexts"], case["tokens"]
    part = [r.uniform(0.25, 2.0) for _ in range(n)]
    got = [max(1, int(total * p / sum(part))) for p in part]
    got[-1] += total - sum(got)
    return got


# ---- inputs --------------------------------------------------------------------------------
class _Inputs:
    """Tensors made on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, shape, mean, std):
        x = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.bfloat16)
        return x.mul_(std).add_(mean) if mean else x.mul_(std)

    def hidden(self, n, d, norm):
        x = torch.randn((n, d), generator=self.g, device="cuda", dtype=torch.bfloat16)
        ch = torch.randperm(d, generator=self.g, device="cuda")[: max(1, round(0.01 * d))]
        x[:, ch] *= 20
        return x.add_(0.25) if norm == "layer" else x

    def table(self, n_blocks, num_pages):
        return torch.randperm(num_pages, generator=self.g, device="cuda")[:n_blocks].to(torch.int32)


def _pages(n_blocks):
    return max(n_blocks * 5 // 4, n_blocks + 1)


def _weights(case, inp):
    """One layer's projection [K rows | V rows], gain, shift and bias (None where the width has none)."""
    d, heads, hd, _, _, norm = WIDTHS[case["width"]]
    w = inp.normal((2 * heads * hd, d), 0.0, 0.02)
    gain = inp.normal((d,), 1.0, 0.1)
    shift = inp.normal((d,), 0.0, 0.05) if norm == "layer" else None
    bias = inp.normal((2 * heads * hd,), 0.0, 0.05) if norm != "rms" else None
    return w, gain, shift, bias


def _context(case, inp, max_position, num_pages):
    d, heads, hd, theta, style, norm = WIDTHS[case["width"]]
    ctx = hc.Context(hc.ModelDesc(case["layers"], d, heads, heads, hd, BLOCK, max_position, style, theta, 1e-5,
                                  hc.HC_NORM_LAYER if norm == "layer" else hc.HC_NORM_RMS))
    stream = torch.cuda.current_stream().cuda_stream
    pools = []
    for l in range(case["layers"]):
        pool = torch.zeros((num_pages, 2, BLOCK, heads, hd), dtype=torch.bfloat16, device="cuda")
        ctx.set_kv_pool(l, pool, num_pages)
        pools.append(pool)
        w, gain, shift, bias = _weights(case, inp)
        if norm == "rms":
            ctx.set_layer_weights(l, w, gain, stream)
        else:
            ctx.set_layer_weights_affine(l, w, gain, shift, bias, stream)
        torch.cuda.synchronize()       # the weights' buffers are reused from here on
    return ctx, pools


def _places(case, inp):
    """Positions, block tables and (a batch) row offsets, the pool's pages and the positions there are."""
    path, n = case["path"], case["tokens"]
    s = {}
    if path == "ragged":
        lens = lengths(case)
        blocks = [-(-k // BLOCK) for k in lens]
        num_pages = _pages(sum(blocks))
        perm = inp.table(sum(blocks), num_pages)
        s["table"] = torch.full((len(lens), max(blocks)), -1, dtype=torch.int32, device="cuda")
        at = 0
        for i, b in enumerate(blocks):
            s["table"][i, :b] = perm[at:at + b]
            at += b
        s["cu"] = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
        s["positions"] = torch.from_numpy(np.concatenate([np.arange(k, dtype=np.int32) for k in lens])).cuda()
        s["contexts"], s["blocks"], top = len(lens), max(blocks), max(lens)
    else:
        top = case["offset"] + n
        s["blocks"] = -(-top // BLOCK)
        places = 2 if path == "rows" else 1               # a context comes back into other pages
        num_pages = _pages(places * s["blocks"])
        perm = inp.table(places * s["blocks"], num_pages)
        s["table"] = perm[:s["blocks"]].clone()
        if path == "rows":
            s["other_table"] = perm[s["blocks"]:].clone()
        s["positions"] = torch.arange(case["offset"], top, dtype=torch.int32, device="cuda")
    return s, num_pages, top


def prepare(case, seed):
    inp = _Inputs(seed)
    d, heads, hd, _, _, norm = WIDTHS[case["width"]]
    path, n = case["path"], case["tokens"]
    if path == "save":
        return _prepare_save(case, inp, d)
    s, num_pages, top = _places(case, inp)
    s["path"], s["n"] = path, n
    s["ctx"], s["pools"] = _context(case, inp, top, num_pages)
    if path == "rows":
        s["pools"][0].normal_(generator=inp.g)
        s["rows"] = torch.zeros((n, 2 * heads * hd), dtype=torch.bfloat16, device="cuda")
    elif path == "store":
        chunks = -(-top // CHUNK)
        s["offset"] = case["offset"]
        s["copy"] = torch.cuda.Stream()
        s["store"] = hc.Store(case["layers"], d, CHUNK, (chunks + 1) * case["layers"])
        for l in range(case["layers"]):
            s["store"].append(7, l, inp.hidden(top, d, norm).view(torch.int16).cpu().numpy(), top)
    else:
        s["hidden"] = [inp.hidden(n, d, norm) for _ in range(case["layers"])]
    return s


def _prepare_save(case, inp, d):
    n, decoding, layers = case["tokens"], case["contexts"], case["layers"]
    rows = n + decoding
    store = hc.Store(layers, d, CHUNK, (-(-n // CHUNK) + decoding + 1) * layers)
    s = {"path": "save", "rows": rows, "layers": layers, "d": d, "store": store, "contexts": list(range(decoding + 1)), "saved": False}
    s["saver"] = hc.Saver(store, rows, n_slots=4, n_threads=8)
    s["down"] = torch.cuda.Stream()
    s["row_context"] = np.concatenate([np.zeros(n, np.int64), np.arange(1, decoding + 1, dtype=np.int64)])
    s["hidden"] = [inp.hidden(rows, d, "rms") for _ in range(layers)]
    return s


# ---- one pass --------------------------------------------------------------------------------
def run(s):
    ctx, path = s.get("ctx"), s["path"]
    stream = torch.cuda.current_stream().cuda_stream
    if path == "layer":
        ctx.restore_kv(0, s["hidden"][0], s["positions"], s["n"], s["table"], s["blocks"], stream)
    elif path == "layers":
        ctx.restore_kv_layers(0, s["hidden"], s["positions"], s["n"], s["table"], s["blocks"], stream)
    elif path == "ragged":
        ctx.restore_kv_ragged(0, s["hidden"][0], s["positions"], s["n"], s["cu"], s["contexts"], s["table"], s["blocks"], stream)
    elif path == "store":
        ctx.restore_context(s["store"], 7, s["offset"], s["n"], 0, s["table"], s["blocks"], stream, s["copy"].cuda_stream)
    elif path == "rows":
        ctx.gather_kv(0, s["rows"], s["positions"], s["n"], s["table"], s["blocks"], stream)
        ctx.scatter_kv(0, s["rows"], s["positions"], s["n"], s["other_table"], s["blocks"], stream)
        return [s["rows"], s["pools"][0]]
    else:
        return _run_save(s, stream)
    return s["pools"]


def _run_save(s, stream):
    store, saver = s["store"], s["saver"]
    if s["saved"]:                     # the conversations of the pass before have ended
        for c in s["contexts"]:
            store.drop(c)
    s["saved"] = True
    for l, x in enumerate(s["hidden"]):
        saver.save_layer_deferred(l, x, s["rows"], s["row_context"], stream, s["down"].cuda_stream)
    saver.fence(stream)
    saver.flush()
    torch.cuda.current_stream().synchronize()
    out = []
    for l in range(s["layers"]):
        for c in s["contexts"]:
            for k in range(-(-store.tokens(c, l) // CHUNK)):
                at, rows = store.chunk(c, l, k)
                chunk = (ctypes.c_uint16 * (rows * s["d"])).from_address(at)
                chunk.store = store        # the array reads the store's memory: it keeps the store alive
                out.append(np.frombuffer(chunk, dtype=np.uint16))
    return out


# ---- what a pass cannot do without, and how far two correct ones may differ --------------------
def work(case):
    d, heads, hd, _, style, norm = WIDTHS[case["width"]]
    d_kv, n = heads * hd, case["tokens"]
    if case["path"] == "save":         # every row read on the device and written on the host
        return {"bytes": 2 * case["layers"] * (n + case["contexts"]) * 2 * d, "flops": 0}
    if case["path"] == "rows":         # read and written by the gather, and again by the scatter
        return {"bytes": 4 * n * 2 * d_kv * 2, "flops": 0}
    layer = n * d * 2 + 2 * d_kv * d * 2 + n * 2 * d_kv * 2
    if style != 2:
        layer += n * hd * 4            # (cos, sin) rows
    if norm != "rms":
        layer += 2 * d_kv * 8          # additive constants
    if case["path"] == "store":
        layer += 2 * n * d * 2         # read from the host, written to the device
    return {"bytes": case["layers"] * layer, "flops": case["layers"] * 4 * n * d * d_kv}


def tolerance(case):
    if case["path"] in ("rows", "save"):
        return "exact"
    # bf16 results of 32-bit sums over bf16 products: 2.3e-3 off the 64-bit values, of which half is the
    # rounding of the gain-folded weights and half that of the results
    return {"rel": 0.01, "max": 0.05}


# ---- the same in 64 bits ---------------------------------------------------------------------
def exact(case, seed):
    """What `run` returns, in plain torch with 64-bit inputs, sums and results: normalisation,
    K|V projection, rotation of K, rows into their pages."""
    path, n = case["path"], case["tokens"]
    if path in ("rows", "save"):       # bytes that are moved
        return None
    inp = _Inputs(seed)
    d, heads, hd, theta, style, norm = WIDTHS[case["width"]]
    s, num_pages, top = _places(case, inp)
    weights = [_weights(case, inp) for _ in range(case["layers"])]
    pos = s["positions"].long()
    if path == "ragged":
        context = torch.repeat_interleave(torch.arange(s["contexts"], device="cuda"), s["cu"].long().diff())
        page = s["table"][context, pos // BLOCK].long()
    else:
        page = s["table"][pos // BLOCK].long()
    half = torch.arange(hd // 2, dtype=torch.float64, device="cuda")
    angle = pos.double()[:, None] * theta ** (-2 * half / hd)
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]
    out = []
    for w, gain, shift, bias in weights:
        x = inp.hidden(top if path == "store" else n, d, norm)[-n:].double()
        if norm == "layer":
            x -= x.mean(1, keepdim=True)
        x *= (x.square().mean(1, keepdim=True) + 1e-5).rsqrt()
        x *= gain.double()
        if shift is not None:
            x += shift.double()
        y = x @ w.double().t()
        if bias is not None:
            y += bias.double()
        k, v = y.view(n, 2, heads, hd).unbind(1)
        if style != 2:
            a, b = (k[..., :hd // 2], k[..., hd // 2:]) if style == 0 else (k[..., 0::2], k[..., 1::2])
            a, b = a * cos - b * sin, b * cos + a * sin
            k = torch.cat([a, b], -1) if style == 0 else torch.stack([a, b], -1).flatten(-2)
        pool = torch.zeros((num_pages, 2, BLOCK, heads, hd), dtype=torch.float64, device="cuda")
        pool[page, 0, pos % BLOCK] = k
        pool[page, 1, pos % BLOCK] = v
        out.append(pool)
    return out
