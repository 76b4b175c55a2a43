"""The work that users of this framework have it do, as cases that can be timed.

Four operations, all through the package's public entry points:

  forward   kan_vq_layer_forward / kan_vq_head_forward / kan_vq_head_forward_static: a head of
            one to three VQ-KAN layers, or a group of heads on one input
  dense     kan_dense_layer_forward: the layer before compression
  assign    kan_vq_assign: the compression step (nearest codebook shape of every edge)

A case is a dict of plain values.  Keys of a forward case:

  widths    "2048-1024-256": inputs, hidden widths, outputs of each head
  heads     number of heads that share the input
  batch     samples per call
  K         codebook rows per layer; index type u16 up to 65,536, u32 above
  codebook  "f32" | "f16" | "i8" | "bfp8"        gains  "f16" | "f32" | "q8" (one byte, i8 only)
  rule      "bspline" (cubic) | "pli" (two-tap)  path   "auto" | "precise" | "fp16"
  use       "uniform" | "zipf": how the edges spread over the codebook
  prepared  whether the program regrouped its layers once after loading (batch <= 4 profits)
  buffers   "kept": workspace and output live as long as the program (a server's loop);
            "plain": y = forward(heads, x), the call brings its own; "static": the entry point
            with the library's own scratch, output kept
"""
import math

import torch

from paper_2512_15742_amd import binding as kb
from paper_2512_15742_amd import synth

# The widest layer that a case may have, and the most edge evaluations (edges x samples) of a
# forward or dense case: one 4096 x 4096 layer at batch 8192.
MOST_EVALS = 4096 * 4096 * 8192


def _forward(name, widths, batch, K=65536, *, heads=1, codebook="i8", gains="f16", rule="bspline", path="auto",
             use="uniform", prepared=False, buffers="kept"):
    return {"name": name, "op": "forward", "widths": widths, "heads": heads, "batch": batch, "K": K,
            "codebook": codebook, "gains": gains, "rule": rule, "path": path, "use": use, "prepared": prepared,
            "buffers": buffers}


def listed():
    return [
        # The smallest configuration, called the short way: a notebook, a unit test, a tiny KAN.
        _forward("layer 64-32, batch 16", "64-32", 16, 256, codebook="f32", gains="f32", buffers="plain"),
        # Serving one request at a time from the two-layer Int8 head, layers regrouped once at load time.
        _forward("head, batch 1, prepared", "2048-1024-256", 1, prepared=True),
        # The same head in the four-bytes-per-edge format of the paper, under a caller that may not
        # allocate: a captured graph, an embedded loop.
        _forward("head q8, batch 4, static", "2048-1024-256", 4, gains="q8", buffers="static"),
        # Small dynamic batches of a server on the layers as given.
        _forward("head, batch 16", "2048-1024-256", 16),
        # The largest layer at low batch: the one whose parameter stream fills the memory system.
        _forward("layer 4096-4096, batch 2", "4096-4096", 2, 262144, prepared=True),
        # Widths that come from a data set and not from a tile size; two-tap rule, fp16 codebook, the
        # assignment histogram of a trained layer.
        _forward("ragged head, batch 37", "1000-333-21", 37, 5000, codebook="f16", gains="f32", rule="pli", use="zipf",
                 buffers="plain"),
        # Many task heads on one backbone feature.
        _forward("50 heads, batch 64", "2048-256-21", 64, heads=50),
        # Backbone feature layer with the fp32 codebook, evaluated at full precision (validation).
        _forward("layer 2048-512, batch 256", "2048-512", 256, codebook="f32", gains="f32", path="precise", buffers="plain"),
        # The headline: throughput inference of the head.
        _forward("head, batch 1024", "2048-1024-256", 1024),
        # Offline evaluation of the largest layer, the largest batch.
        _forward("layer 4096-4096, batch 8192", "4096-4096", 8192, 262144),
        # The layer before compression, at a server's batch.
        {"name": "dense 2048-512, batch 16", "op": "dense", "widths": "2048-512", "batch": 16, "buffers": "kept"},
        # Compressing one trained layer against its codebook.
        {"name": "assign 2048-512", "op": "assign", "widths": "2048-512", "K": 65536},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A width between lo and hi: half of them whole multiples of 32, the others as they fall."""
    n = _log_int(rng, lo, hi)
    return min(hi, max(32, (n + 16) // 32 * 32)) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["head"] * 6 + ["heads"] * 2 + ["dense"] * 2 + ["assign"] * 2)
    if kind == "assign":
        return {"op": "assign", "widths": "%d-%d" % (_width(rng, 64, 2048), _width(rng, 32, 512)),
                "K": rng.choice([256, 65536, _log_int(rng, 256, 65536)])}
    if kind == "dense":
        return {"op": "dense", "widths": "%d-%d" % (_width(rng, 64, 2048), _width(rng, 32, 512)),
                "batch": _log_int(rng, 1, 1024), "buffers": rng.choice(["kept", "plain"])}
    path = rng.choice(["auto", "auto", "auto", "precise", "fp16"])
    if kind == "heads":
        widths = [_width(rng, 256, 2048), _width(rng, 64, 256), rng.choice([21, _log_int(rng, 4, 128)])]
        heads, batch = _log_int(rng, 2, 50), _log_int(rng, 1, 128)
        K = rng.choice([65536, _log_int(rng, 1024, 65536)])
    else:
        layers = rng.choice([1, 2, 2, 3])
        top = 4096 if layers == 1 else 2048
        widths = [_width(rng, 64, top), _width(rng, 32, top if layers == 1 else 1024)]
        while len(widths) <= layers:
            widths.append(_width(rng, 16, widths[-1]) if len(widths) < layers else _log_int(rng, 8, max(8, widths[-1])))
        heads, edges = 1, sum(a * b for a, b in zip(widths, widths[1:]))
        most = MOST_EVALS // (4 if path == "precise" else 1)      # (fp32-grade products cost three to four times as much)
        batch = _log_int(rng, 1, min(8192, most // edges))
        K = rng.choice([65536, _log_int(rng, 256, 65536), 262144 if edges >= 1 << 22 else 65536])
    codebook = rng.choice(["i8", "i8", "i8", "f16", "f32", "bfp8"])
    gains = rng.choice(["f16", "f16", "f32"] + (["q8"] if codebook == "i8" else []))
    case = _forward("", "-".join(map(str, widths)), batch, K, heads=heads, codebook=codebook, gains=gains,
                    rule=rng.choice(["bspline", "bspline", "bspline", "pli"]),
                    path=path, use=rng.choice(["uniform", "uniform", "zipf"]),
                    prepared=batch <= 4 and rng.random() < 0.6,
                    buffers=rng.choice(["kept", "kept", "plain"] + (["static"] if batch <= 16 and heads == 1 and
                                                                    len(widths) > 2 else [])))
    del case["name"]
    return case


# ---- inputs, drawn on the GPU with the distributions of the package's own generator ----------------


def _shapes(g, K):
    """K zero-mean unit-norm rows of ten numbers."""
    s = torch.randn((K, 10), generator=g, device="cuda")
    s -= s.mean(1, keepdim=True)
    return s / s.norm(dim=1, keepdim=True)


def _layer(g, case, n_in, n_out):
    K = case["K"]
    shapes, scale = _shapes(g, K), 1.0
    if case["codebook"] == "i8":
        scale = float(shapes.abs().max()) / 127.0
        codebook = (shapes / scale).round().clamp(-127, 127).to(torch.int8).cpu().numpy()
    elif case["codebook"] == "bfp8":
        codebook = synth.quantise_shapes_bfp8(shapes.cpu().numpy())
    else:
        codebook = shapes.to(torch.float16 if case["codebook"] == "f16" else torch.float32).cpu().numpy()
    if case["use"] == "zipf":   # P(rank r) ~ 1 / r, the ranks scattered over the codebook
        upto = (1.0 / torch.arange(1, K + 1, device="cuda", dtype=torch.float64)).cumsum(0)
        u = torch.rand(n_in * n_out, generator=g, device="cuda", dtype=torch.float64) * upto[-1]
        ranks = torch.searchsorted(upto, u).clamp_(max=K - 1)
        idx = torch.randperm(K, generator=g, device="cuda")[ranks].view(n_in, n_out)
    else:
        idx = torch.randint(0, K, (n_in, n_out), generator=g, device="cuda")
    idx = idx.to(torch.int32).cpu().numpy().view("uint32")
    gain = torch.randn((n_in, n_out), generator=g, device="cuda").abs_().mul_(0.1)
    bias = torch.randn((n_in, n_out), generator=g, device="cuda").mul_(0.01)
    params = None
    if case["gains"] == "q8":
        gain, bias, params = synth.encode_gain_bias_q8(gain.cpu().numpy(), bias.cpu().numpy())
    else:
        dt = torch.float16 if case["gains"] == "f16" else torch.float32
        gain, bias = gain.to(dt).cpu().numpy(), bias.to(dt).cpu().numpy()
    p = synth.VQLayerParams(n_in, n_out, K, codebook, scale, idx.astype("uint16") if K <= 65536 else idx, gain, bias, params)
    layer = kb.VQLayer(p, rule=kb.KAN_RULE_PLI2 if case["rule"] == "pli" else kb.KAN_RULE_BSPLINE3)
    return layer.prepare() if case["prepared"] else layer


def _widths(case):
    return [int(w) for w in case["widths"].split("-")]


def _x(g, batch, n_in):
    return torch.rand((batch, n_in), generator=g, device="cuda").mul_(2.0).sub_(1.0)


PATHS = {"auto": kb.KAN_PATH_AUTO, "precise": kb.KAN_PATH_GATHER, "fp16": kb.KAN_PATH_MFMA}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    w = _widths(case)
    if case["op"] == "assign":
        # trained grids: gain * shape + bias with five per cent of noise
        shapes = _shapes(g, case["K"])
        k = torch.randint(0, case["K"], (w[0], w[1]), generator=g, device="cuda")
        gain = torch.randn((w[0], w[1], 1), generator=g, device="cuda").abs_().mul_(0.1).add_(1e-3)
        bias = torch.randn((w[0], w[1], 1), generator=g, device="cuda").mul_(0.01)
        noise = torch.randn((w[0], w[1], 10), generator=g, device="cuda").mul_(0.05)
        return {"run": _run_assign, "coef": (gain * (shapes[k] + noise) + bias).contiguous(), "codebook": shapes}
    if case["op"] == "dense":
        s = {"run": _run_dense, "x": _x(g, case["batch"], w[0]), "ws": None, "y": None,
             "coef": torch.randn((w[0], w[1], 10), generator=g, device="cuda").mul_(0.03)}
        if case["buffers"] == "kept":
            s["y"] = torch.empty((case["batch"], w[1]), device="cuda")
            s["ws"] = torch.empty(max(256, kb.kan_dense_workspace_bytes(w[0], w[1], case["batch"])), dtype=torch.uint8, device="cuda")
        return s
    heads = [[_layer(g, case, a, b) for a, b in zip(w, w[1:])] for _ in range(case["heads"])]
    path, one = PATHS[case["path"]], case["heads"] == 1 and len(w) == 2
    s = {"run": _run_static if case["buffers"] == "static" else _run_layer if one else _run_head, "heads": heads,
         "layer": heads[0][0], "x": _x(g, case["batch"], w[0]), "path": path, "ws": None, "y": None}
    if case["buffers"] != "plain":
        shape = (case["batch"], w[-1]) if s["run"] is _run_layer else (case["heads"], case["batch"], w[-1])
        s["y"] = torch.empty(shape, device="cuda")
    if case["buffers"] == "kept":
        s["ws"] = torch.empty(max(256, kb.kan_vq_workspace_bytes(heads, case["batch"], path)), dtype=torch.uint8, device="cuda")
    return s


# ---- one pass ---------------------------------------------------------------------------------------


def _run_layer(s):
    return kb.kan_vq_layer_forward(s["layer"], s["x"], path=s["path"], ws=s["ws"], y=s["y"])


def _run_head(s):
    return kb.kan_vq_head_forward(s["heads"], s["x"], path=s["path"], ws=s["ws"], y=s["y"])


def _run_static(s):
    return kb.kan_vq_head_forward_static(s["heads"], s["x"], path=s["path"], y=s["y"])


def _run_dense(s):
    return kb.kan_dense_layer_forward(s["coef"], s["x"], ws=s["ws"], y=s["y"])


def _run_assign(s):
    return kb.kan_vq_assign(s["coef"], s["codebook"])


def run(state):
    return state["run"](state)


# ---- what a pass cannot do without, and how close another correct one comes --------------------------


def work(case):
    w = _widths(case)
    edges = sum(a * b for a, b in zip(w, w[1:]))
    if case["op"] == "assign":
        idx = 2 if case["K"] <= 65536 else 4
        return {"bytes": edges * (40 + idx + 8) + 40 * case["K"], "flops": 20 * edges * case["K"]}
    b = case["batch"]
    if case["op"] == "dense":
        return {"bytes": 40 * edges + 4 * b * (w[0] + w[1]), "flops": 8 * edges * b}
    per_edge = (2 if case["K"] <= 65536 else 4) + {"f16": 4, "f32": 8, "q8": 2}[case["gains"]]
    row = {"f32": 40, "f16": 20, "i8": 10, "bfp8": 12}[case["codebook"]]
    layers = len(w) - 1
    return {"bytes": case["heads"] * (edges * per_edge + layers * case["K"] * row + 4 * b * w[-1]) + 4 * b * w[0],
            "flops": case["heads"] * edges * b * (8 if case["rule"] == "bspline" else 4)}


def tolerance(case):
    if case["op"] == "assign":
        return {"rel": 1e-5, "differ": 1e-4}     # gains and biases in fp32; ids but for near ties
    if case["op"] == "forward" and (case["path"] == "fp16" or (case["path"] == "auto" and case["batch"] >= 32)):
        return {"rel": 3e-3}                     # fp16 operands (2^-11), fp32 sums, up to three layers
    return {"rel": 1e-5}                         # fp32-grade sums
