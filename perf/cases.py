"""Measured work of the library: the calls a decoding program makes, over the sizes it makes them with.

A case is one pass of one of these kinds:

  step     the cached denoising step of `layers` layers: project the window rows, scatter, attend
           (fc_qkv_project_scatter, fc_active_attention), every layer on its own input
  refresh  the projections of a wide region and its attention (fc_refresh): the initial pass over a
           prompt, or the periodic refresh of the generation region
  layer    `layers` whole layers chained (fc_full_layer_step), for short windows, batched windows and
           whole prompts
  unmask   the end of a step: final norm, vocabulary projection with arg-max and confidence,
           confidence-ranked fill (fc_rmsnorm, fc_lm_head_argmax, fc_unmask_select)
  accept   guided acceptance of a speculation block on given logits (fc_guided_accept)

Geometries are those of paper_2505_21467_amd.inputs: the small full-precision configuration and its
neighbourhood ("tiny", float32 mostly), and the two bf16 model geometries.  Weights ~ N(0, 0.02),
activations and cached keys / values ~ N(0, 1), as everywhere in this repository.  A program holds one
cache and one set of weights per layer, so passes go over several layers and their weights come from
HBM, not from a cache that the pass before left warm.
"""
import random

import torch

from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs

MASK = 151666  # id of the mask token in the token arrays

# hidden, query heads, kv heads, head_dim, d_ff, eps
GEOMETRY = {
    "dream7b": (3584, 28, 4, 128, 18944, 1e-6),
    "llada8b": (4096, 32, 32, 128, 12288, 1e-5),
}


def _model(name):
    d, hq, hkv, dh, f, eps = GEOMETRY[name]
    return {"dtype": "bf16", "hidden": d, "hq": hq, "hkv": hkv, "dh": dh, "d_ff": f, "eps": eps}


def _tiny(hidden=256, hq=4, hkv=4, dh=64, dtype="f32"):
    return {"dtype": dtype, "hidden": hidden, "hq": hq, "hkv": hkv, "dh": dh, "d_ff": 2 * hidden, "eps": 1e-6}


def _window(kind, model, layers, batch, rows, cached, gen, ragged=False, bias=False):
    """rows: window rows per sequence; the keys are the rows [0, cached + gen), the window starts at `cached`."""
    return dict(model, kind=kind, layers=layers, batch=batch, rows=rows, cached=cached, gen=gen, ragged=ragged, bias=bias)


def _unmask(dtype, hidden, batch, rows, vocab, fill):
    return {"kind": "unmask", "dtype": dtype, "hidden": hidden, "batch": batch, "rows": rows, "vocab": vocab, "fill": fill}


def _accept(batch, rows, masked, vocab, topk, tau):
    return {"kind": "accept", "batch": batch, "rows": rows, "masked": masked, "vocab": vocab, "topk": topk, "tau": tau}


def listed():
    dream, llada = _model("dream7b"), _model("llada8b")
    return [
        # the smallest call: one full-precision layer of the tiny configuration, where launches count
        dict(_window("step", _tiny(), 1, 1, 32, 256, 32), name="step tiny f32"),
        # one user, one block of 32 tokens behind a prompt of 1024: the interactive step
        dict(_window("step", dream, 8, 1, 32, 1024, 32), name="step dream L1024"),
        # the same behind a long document
        dict(_window("step", dream, 8, 1, 32, 16384, 416), name="step dream L16384"),
        # four users of the multi-head geometry, blocks of 64: bound by the keys and values
        dict(_window("step", llada, 2, 4, 64, 4096, 64), name="step llada B4 L4096"),
        # only the rows that are still masked are projected: odd counts, lists padded with -1, biases
        dict(_window("step", dream, 8, 3, 19, 1543, 38, ragged=True, bias=True), name="step dream ragged"),
        # periodic refresh of the generation region of eight sequences
        dict(_window("refresh", dream, 2, 8, 256, 2048, 256), name="refresh dream B8 R256"),
        # whole layers: one block of one user, where every weight matrix is read for 32 rows
        dict(_window("layer", dream, 2, 1, 32, 1024, 32), name="layer dream B1 A32"),
        # whole layers: the blocks of eight users together
        dict(_window("layer", dream, 2, 8, 32, 2048, 256), name="layer dream B8 A32"),
        # whole layers: the initial pass over prompt and generation region of one sequence
        dict(_window("layer", dream, 2, 1, 2304, 0, 2304), name="layer dream prefill"),
        # the end of a step for one block, and for the blocks of eight users
        dict(_unmask("bf16", 3584, 1, 32, 152064, 4), name="unmask B1 A32"),
        dict(_unmask("bf16", 3584, 8, 32, 152064, 4), name="unmask B8 A32"),
        # speculation block of one user against the guide's logits
        dict(_accept(1, 32, 32, 152064, 2, 0.5), name="accept B1 A32"),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over the logarithm."""
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choices(("step", "refresh", "layer", "unmask", "accept"), (5, 2, 4, 2, 1))[0]
    if kind == "accept":
        batch, rows = _log(rng, 1, 4), _log(rng, 4, 64)
        return _accept(batch, rows, rng.randint((rows + 1) // 2, rows), _vocab(rng), rng.randint(1, 8), rng.choice((0.0, 0.5)))
    tiny = rng.random() < 0.25
    if kind == "unmask":
        batch = _log(rng, 1, 8)
        rows = _log(rng, 1, 32)
        if tiny:
            return _unmask("f32", rng.choice((256, 384, 512)), min(batch, 4), rows, _log(rng, 300, 4000), rng.randint(1, 4))
        vocab = _vocab(rng)
        if vocab & 1:  # a small model with a vocabulary of its own
            batch = 1
        return _unmask("bf16", rng.choice((3584, 4096)), batch, rows, vocab, rng.randint(1, 4))
    if tiny:
        hkv, dtype = rng.choice((1, 2, 4)), rng.choice(("f32", "f32", "f32", "bf16"))
        model = _tiny(rng.choice((256, 384, 512)), hkv * rng.choice((1, 2, 4)), hkv, rng.choice((64, 128)), dtype)
    else:
        model = _model(rng.choice(("dream7b", "dream7b", "llada8b")))
    batch = _log(rng, 1, 4 if tiny else 8)
    if kind == "refresh" or (kind == "layer" and rng.random() < 0.4):
        rows = _log(rng, 48, max(48, (160 if tiny else 2304) // batch))
        cached = rng.choice((0, _log(rng, 64, 2048)))  # the whole sequence, or a region behind a prompt
        return _window(kind, model, 2, batch, rows, cached, rows, bias=rng.random() < 0.3)
    rows = _log(rng, 4, 64)
    cached = _log(rng, 64, 2048 if tiny else 16384)
    if not tiny:  # keys and values of a layer: at most those of the largest listed step
        cached = min(cached, 4 * 4096 * 32 // (batch * model["hkv"]))
    ragged = rng.random() < 0.4
    gen = 2 * rows if ragged else rng.choice((rows, rows, rows + _log(rng, 1, 384)))
    layers = rng.randint(1, 4) if tiny else (2 if kind == "layer" or model["hkv"] > 4 else rng.randint(4, 8))
    return _window(kind, model, layers, batch, rows, cached, gen, ragged, rng.random() < 0.3)


def _vocab(rng):
    """The 7B vocabulary, a round one, or any other (odd) size."""
    return rng.choice((152064, 152064, 32000, _log(rng, 1000, 16000) | 1))


class _Cache:
    """A cache handle and its storage, released with the state that holds it."""

    def __init__(self, c, device):
        self.cfg = fc.make_config(c["layers"], c["batch"], c["hidden"], c["hq"], c["hkv"], c["dh"], c["cached"] + c["gen"], c["dtype"])
        n = fc.fc_cache_storage_bytes(self.cfg) // (4 if c["dtype"] == "f32" else 2)
        self.k = torch.zeros(n, dtype=inputs.TORCH_DTYPE[c["dtype"]], device=device)
        self.v = torch.zeros_like(self.k)
        self.handle = fc.fc_cache_alloc(self.cfg, self.k, self.v)

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            fc.fc_cache_free(self.handle)
            self.handle = None


def _positions(c, seed):
    """Window positions of a ragged step: what stays masked of a region twice the window, -1 behind it."""
    rng = random.Random(seed)
    pos = []
    for b in range(c["batch"]):
        n = c["rows"] if b == 0 else rng.randint(1, c["rows"])
        pos.append(sorted(rng.sample(range(c["cached"], c["cached"] + c["gen"]), n)) + [-1] * (c["rows"] - n))
    return torch.tensor(pos, dtype=torch.int32)


def prepare(case, seed):
    c, dev = case, torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    if c["kind"] == "accept":
        return _prepare_accept(c, gen, dev, seed)
    dt = inputs.TORCH_DTYPE[c["dtype"]]

    def rnd(shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=dt, device=dev).normal_(mean, std, generator=gen)

    if c["kind"] == "unmask":
        return _prepare_unmask(c, rnd, gen, dev, seed)
    n, d, e = c["layers"], c["hidden"], c["hq"] * c["dh"]
    width = (c["hq"] + 2 * c["hkv"]) * c["dh"]
    s = {"case": c, "cache": _Cache(c, dev), "kv_len": c["cached"] + c["gen"]}
    shape = (c["batch"], c["hkv"], s["kv_len"], c["dh"])
    for layer in range(n):
        fc.fc_cache_write_rows(s["cache"].handle, layer, rnd(shape), rnd(shape), 0, s["kv_len"])
    s["pos"] = _positions(c, seed).to(dev) if c["ragged"] else None
    s["w_qkv"] = [rnd((width, d), 0.02) for _ in range(n)]
    s["b_qkv"] = [rnd((width,), 0.02) if c["bias"] else None for _ in range(n)]
    if c["kind"] == "layer":
        s["x"] = rnd((c["batch"], c["rows"], d))
        s["y"] = [torch.empty_like(s["x"]) for _ in range(2)]
        s["tensors"] = []  # the weights structs hold pointers only
        s["weights"] = []
        for layer in range(n):
            t = {"norm1": rnd((d,), 0.1, 1.0), "w_qkv": s["w_qkv"][layer], "b_qkv": s["b_qkv"][layer], "w_out": rnd((d, e), 0.02),
                 "norm2": rnd((d,), 0.1, 1.0), "w_gate": rnd((c["d_ff"], d), 0.02), "w_up": rnd((c["d_ff"], d), 0.02),
                 "w_down": rnd((d, c["d_ff"]), 0.02)}
            s["tensors"].append(t)
            s["weights"].append(fc.make_layer_weights(d_ff=c["d_ff"], eps=c["eps"], **t))
        s["ws_bytes"] = fc.fc_full_layer_workspace_bytes(s["cache"].cfg, c["d_ff"], c["rows"])
    else:
        s["x"] = rnd((n, c["batch"], c["rows"], d))
        s["q"] = torch.zeros((n, c["batch"], c["hq"], c["rows"], c["dh"]), dtype=dt, device=dev)
        s["o"] = torch.zeros((n, c["batch"], c["rows"], e), dtype=dt, device=dev)
        s["x_l"], s["q_l"], s["o_l"] = list(s["x"]), list(s["q"]), list(s["o"])
        s["ws_bytes"] = fc.fc_workspace_bytes(s["cache"].cfg, c["rows"])
    s["ws"] = torch.empty(max(16, s["ws_bytes"]), dtype=torch.uint8, device=dev)
    return s


def _prepare_unmask(c, rnd, gen, dev, seed):
    m, d, v = c["batch"] * c["rows"], c["hidden"], c["vocab"]
    s = {"case": c, "w_vocab": rnd((v, d), 0.02), "norm": rnd((d,), 0.1, 1.0), "seq_len": 4 * c["rows"]}
    # hidden states that lean towards one token each, some more than others: confidences from low to high
    lean = torch.randint(0, v, (m,), generator=gen, device=dev)
    force = torch.empty((m, 1), device=dev).uniform_(3.0, 12.0, generator=gen)
    s["x"] = (rnd((m, d)).float() + force * s["w_vocab"][lean].float()).to(s["norm"].dtype)
    s["h"] = torch.empty_like(s["x"])
    s["tok"] = torch.zeros(m, dtype=torch.int32, device=dev)
    s["conf"] = torch.zeros(m, dtype=torch.float32, device=dev)
    s["ws_bytes"] = fc.fc_lm_head_workspace_bytes(c["dtype"], m, d, v)
    s["ws"] = torch.empty(max(16, s["ws_bytes"]), dtype=torch.uint8, device=dev)
    _token_arrays(s, c, c["rows"], seed, dev)
    return s


def _prepare_accept(c, gen, dev, seed):
    shape = (c["batch"], c["rows"], c["vocab"])
    s = {"case": c, "seq_len": 4 * c["rows"]}
    # the guide mostly agrees with the diffusion model: a prefix is accepted, then the two part
    s["dlm"] = torch.empty(shape, device=dev).normal_(0.0, 3.0, generator=gen)
    s["ar"] = torch.empty(shape, device=dev).normal_(0.0, 0.3, generator=gen).add_(s["dlm"])
    s["n_accept"] = torch.zeros(c["batch"], dtype=torch.int32, device=dev)
    s["ws_bytes"] = fc.fc_guided_accept_workspace_bytes(c["batch"], c["rows"], c["vocab"])
    s["ws"] = torch.empty(max(16, s["ws_bytes"]), dtype=torch.uint8, device=dev)
    _token_arrays(s, c, c["masked"], seed, dev)
    return s


def _token_arrays(s, c, masked, seed, dev):
    """Token arrays whose window holds `masked` masked positions, and the buffers of the rows that stay masked."""
    rng = random.Random(seed)
    s["start"] = s["seq_len"] - c["rows"]
    tokens = [[rng.randrange(MASK) for _ in range(s["seq_len"])] for _ in range(c["batch"])]
    for row in tokens:
        for a in rng.sample(range(c["rows"]), masked):
            row[s["start"] + a] = MASK
    s["tokens_in"] = torch.tensor(tokens, dtype=torch.int32).to(dev)
    s["tokens"] = s["tokens_in"].clone()
    s["pos_next"] = torch.zeros((c["batch"], c["rows"]), dtype=torch.int32, device=dev)
    s["count_next"] = torch.zeros(c["batch"], dtype=torch.int32, device=dev)


def run(s):
    return _RUN[s["case"]["kind"]](s)


def _run_step(s):
    c, handle = s["case"], s["cache"].handle
    rows, start, kv_len, pos, ws, ws_bytes = c["rows"], c["cached"], s["kv_len"], s["pos"], s["ws"], s["ws_bytes"]
    for layer in range(c["layers"]):
        q = s["q_l"][layer]
        fc.fc_qkv_project_scatter(handle, layer, s["x_l"][layer], s["w_qkv"][layer], s["b_qkv"][layer], start, rows, pos, q)
        fc.fc_active_attention(handle, layer, q, rows, kv_len, pos, s["o_l"][layer], ws, ws_bytes)
    return {"q": s["q"], "o": s["o"], "k": s["cache"].k, "v": s["cache"].v}


def _run_refresh(s):
    c, handle = s["case"], s["cache"].handle
    for layer in range(c["layers"]):
        fc.fc_refresh(handle, layer, s["x_l"][layer], s["w_qkv"][layer], s["b_qkv"][layer], c["cached"], c["rows"], s["kv_len"],
                      s["q_l"][layer], s["o_l"][layer], s["ws"], s["ws_bytes"])
    return {"q": s["q"], "o": s["o"], "k": s["cache"].k, "v": s["cache"].v}


def _run_layer(s):
    c, handle, x = s["case"], s["cache"].handle, s["x"]
    for layer in range(c["layers"]):
        y = s["y"][layer & 1]
        fc.fc_full_layer_step(handle, layer, s["weights"][layer], x, c["cached"], c["rows"], s["pos"], s["kv_len"], y, s["ws"],
                              s["ws_bytes"])
        x = y
    return {"y": x, "k": s["cache"].k, "v": s["cache"].v}


def _run_unmask(s):
    c = s["case"]
    m, d = c["batch"] * c["rows"], c["hidden"]
    s["tokens"].copy_(s["tokens_in"])  # the sequences as they stand at this step
    fc.fc_rmsnorm(c["dtype"], s["x"], s["norm"], 1e-6, m, d, s["h"])
    fc.fc_lm_head_argmax(c["dtype"], s["h"], s["w_vocab"], m, d, c["vocab"], s["tok"], s["conf"], s["ws"], s["ws_bytes"])
    fc.fc_unmask_select(s["tok"], s["conf"], None, s["start"], c["batch"], c["rows"], c["fill"], MASK, s["tokens"], s["seq_len"],
                        s["pos_next"], s["count_next"])
    return {k: s[k] for k in ("tok", "conf", "tokens", "pos_next", "count_next")}


def _run_accept(s):
    c = s["case"]
    s["tokens"].copy_(s["tokens_in"])
    fc.fc_guided_accept(s["dlm"], s["ar"], None, s["start"], c["batch"], c["rows"], c["vocab"], c["topk"], c["tau"], MASK, s["tokens"],
                        s["seq_len"], s["n_accept"], s["pos_next"], s["count_next"], s["ws"], s["ws_bytes"])
    return {k: s[k] for k in ("tokens", "n_accept", "pos_next", "count_next")}


_RUN = {"step": _run_step, "refresh": _run_refresh, "layer": _run_layer, "unmask": _run_unmask, "accept": _run_accept}


def work(case):
    """What one pass cannot do without: inputs read once, outputs written once, products multiplied out."""
    c = case
    if c["kind"] == "accept":
        read = 2 * c["batch"] * c["masked"] * c["vocab"] * 4
        return {"bytes": read + c["batch"] * 32 * c["rows"], "flops": 0}
    es = 4 if c["dtype"] == "f32" else 2
    m = c["batch"] * c["rows"]
    if c["kind"] == "unmask":
        return {"bytes": es * (c["vocab"] * c["hidden"] + m * c["hidden"] + c["hidden"]) + 48 * m,
                "flops": 2 * m * c["hidden"] * c["vocab"]}
    d, e, kv = c["hidden"], c["hq"] * c["dh"], c["hkv"] * c["dh"]
    keys = c["cached"] + c["gen"]
    w = d * (e + 2 * kv)
    elems = w + 2 * c["batch"] * keys * kv + 2 * m * kv + 2 * m * d   # weights, keys and values, the fresh rows, x and y
    flops = 2 * m * w + 4 * m * keys * e
    if c["kind"] == "layer":
        more = d * e + 3 * d * c["d_ff"]
        elems += more + 2 * d
        flops += 2 * m * more
        # rows between two layers need not leave the chip
        return {"bytes": es * (c["layers"] * (elems - 2 * m * d) + 2 * m * d), "flops": c["layers"] * flops}
    elems += 2 * m * e - m * d                                        # q and o instead of y
    return {"bytes": es * c["layers"] * elems, "flops": c["layers"] * flops}


def tolerance(case):
    if case["kind"] == "accept":
        return "exact"  # comparisons of given numbers
    if case["kind"] == "unmask":
        # confidences of logits that are sums over bf16 rows (a row rounded the other way moves a logit by
        # about 1e-4), or over float32 rows; tokens may differ where two logits tie to within that
        return {"rel": 1e-3 if case["dtype"] == "bf16" else 2e-5, "max": 1e-2 if case["dtype"] == "bf16" else 2e-4, "differ": 0.01}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1 if case["kind"] != "layer" else 0.2}
