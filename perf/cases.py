"""The work whose speed this framework answers for: cases over its public entry points, and how to make and run them.

A case is a dict of plain values; lists of per-job numbers are texts ("8,16,32").  Tensors are drawn on the device from
the seed alone with the distributions of the benchmark's workloads: activations and upstream gradients N(0, 1),
backbone weights N(0, 0.02) (N(0, 1 / d_in) inside a block, where the residual stream must keep unit scale),
A_j U(+-1 / sqrt(d_in)), B_j N(0, 0.01).

kind       one pass
"layer"    tlora_fwd, then tlora_bwd with the forward's S reused, of each projection in `dims`
"noalloc"  tlora_fwd_noalloc of one projection (serving loop: no workspace, no backward)
"nano"     tlora_fwd_nano, tlora_bwd_nano over `n_nano` nano-batches of whole `granule`-token sequences
"indexed"  tlora_fwd_indexed, tlora_bwd_indexed; runs of `granule` tokens of the jobs lie shuffled in the batch
"mlp"      tlora_mlp_fwd, tlora_mlp_bwd
"decoder"  tlora_layer_fwd, tlora_layer_bwd
"attention" tlora_attention_fwd, tlora_attention_bwd
"adamw"    tlora_adamw_step over every adapter tensor of the projections in `dims`
"""
import math

import torch

from paper_2602_07263_amd import tlora
from paper_2602_07263_amd import workloads as wk

HEAD_DIM = 128
GATE_UP_DOWN = "4096x12288,4096x12288,12288x4096"


def _ints(text):
    return [int(v) for v in text.split(",")]


def _text(values):
    return ",".join(str(v) for v in values)


def _dims(case):
    return [tuple(int(v) for v in d.split("x")) for d in case["dims"].split(",")]


def _offsets(tokens):
    out = [0]
    for t in tokens:
        out.append(out[-1] + t)
    return out


def listed():
    c2, c3, c4 = wk.config(2), wk.config(3), wk.config(4)
    return [
        # the fp32 configuration (benchmark's 0th): two small jobs; the smallest training call there is
        {"name": "f32_tiny", "kind": "layer", "dtype": "f32", "dims": "256x256", "ranks": "4,8", "tokens": "64,64"},
        # one step of a serving loop that cannot allocate: a few new tokens of each of eight adapters
        {"name": "serve_61_tokens", "kind": "noalloc", "dtype": "bf16", "dims": "4096x4096",
         "ranks": "8,16,32,8,64,16,32,8", "tokens": "1,4,7,1,16,12,11,9"},
        # a fine-tuning job that runs alone: rank 16, one 512-token sequence, the up projection of an 8B-class layer
        {"name": "one_job_512", "kind": "layer", "dtype": "bf16", "dims": "4096x12288", "ranks": "16", "tokens": "512"},
        # four jobs on an attention projection (benchmark's 1st configuration)
        {"name": "attn_proj_7680", "kind": "layer", "dtype": "bf16", "dims": "4096x4096", "ranks": "8,16,32,64",
         "tokens": "2048,1024,4096,512"},
        # the headline: gate, up and down projections of an 8B-class layer, eight jobs (2nd configuration)
        {"name": "mlp_projections_31744", "kind": "layer", "dtype": "bf16", "dims": GATE_UP_DOWN,
         "ranks": _text(c2.ranks), "tokens": _text(c2.tokens)},
        # 32 jobs between 1 and 16384 tokens, ranks 1 to 256, feature sizes of a 14B-class layer (4th configuration)
        {"name": "skewed_32_jobs", "kind": "layer", "dtype": "bf16", "dims": "5120x17408,17408x5120",
         "ranks": _text(c4.ranks), "tokens": _text(c4.tokens)},
        # the gate projection cut into eight nano-batches, as the adaptive controller runs it
        {"name": "nano_8_batches", "kind": "nano", "dtype": "bf16", "dims": "4096x12288", "ranks": _text(c2.ranks),
         "tokens": _text(c2.tokens), "n_nano": 8, "granule": 512},
        # samples of odd lengths of five jobs in arrival order: ragged segments, rows fetched and stored through a list
        {"name": "indexed_ragged_5003", "kind": "indexed", "dtype": "bf16", "dims": "4096x4096",
         "ranks": "3,16,40,8,100", "tokens": "517,1290,801,77,2318", "granule": 37},
        # the MLP half of a layer on a small ragged batch of three jobs
        {"name": "mlp_block_1900", "kind": "mlp", "dtype": "bf16", "d_model": 4096, "d_ff": 12288, "ranks": "8,16,4",
         "tokens": "1024,620,256"},
        # a whole decoder layer on sixteen jobs (3rd configuration), sequences of 2048 tokens; the largest call
        {"name": "decoder_layer_83968", "kind": "decoder", "dtype": "bf16", "d_model": 4096, "d_ff": 12288,
         "heads": 32, "kv_heads": 8, "ranks": _text(c3.ranks), "tokens": _text(c3.tokens), "seq_len": 2048},
        # causal grouped-query attention alone, sequences of 2048 tokens
        {"name": "attention_2048", "kind": "attention", "dtype": "bf16", "heads": 32, "kv_heads": 8, "tokens": "32768",
         "seq_len": 2048},
        # the optimizer step of every adapter of the headline
        {"name": "adamw_48_tensors", "kind": "adamw", "dtype": "bf16", "dims": GATE_UP_DOWN, "ranks": _text(c2.ranks),
         "tokens": "0"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _split(rng, total, jobs):
    """`total` tokens cut at random into at most `jobs` segments of at least one token."""
    jobs = min(jobs, total)
    cuts = sorted(rng.sample(range(1, total), jobs - 1)) if jobs > 1 else []
    return [b - a for a, b in zip([0] + cuts, cuts + [total])]


def _width(rng):
    """A feature size: one of the configurations', or any multiple of 8 between 256 and 16384."""
    if rng.random() < 0.6:
        return rng.choice([1024, 4096, 4096, 5120, 12288, 17408])
    return 8 * _log_uniform(rng, 32, 2048)


def _ranks(rng, n, top=256):
    return [min(top, rng.choice([1, 2, 3, 4, 8, 8, 16, 16, 32, 48, 64, 96, 128, 256])) for _ in range(n)]


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["noalloc"] * 2 + ["nano", "indexed", "mlp", "decoder", "attention", "attention",
                                                         "adamw", "f32"])
    if kind == "f32":
        tok = _split(rng, _log_uniform(rng, 32, 2048), rng.randint(1, 6))
        return {"kind": "layer", "dtype": "f32", "dims": f"{8 * _log_uniform(rng, 16, 128)}x{8 * _log_uniform(rng, 16, 128)}",
                "ranks": _text(_ranks(rng, len(tok), 64)), "tokens": _text(tok)}
    if kind in ("layer", "indexed"):
        tok = _split(rng, _log_uniform(rng, 16, 32768), rng.randint(1, 16))
        case = {"kind": kind, "dtype": "bf16", "dims": f"{_width(rng)}x{_width(rng)}",
                "ranks": _text(_ranks(rng, len(tok))), "tokens": _text(tok)}
        if kind == "indexed":
            case["granule"] = _log_uniform(rng, 1, 512)
        return case
    if kind == "noalloc":
        tok = _split(rng, _log_uniform(rng, 1, 512), rng.randint(1, 12))
        di, do = rng.choice([1024, 2048, 4096]), rng.choice([1024, 2048, 4096, 5120])
        ranks = _ranks(rng, len(tok), 64)
        # what the static scratch holds (16 MiB): packed adapters, per-tile operands, intermediates
        while True:
            R = sum((r + 7) // 8 * 8 for r in ranks)
            if 6 * (R + 32) * (di + do) + (4 * 512 + 512 * 3) * R < (15 << 20):
                break
            ranks = [max(1, r // 2) for r in ranks]
        return {"kind": kind, "dtype": "bf16", "dims": f"{di}x{do}", "ranks": _text(ranks), "tokens": _text(tok)}
    if kind == "nano":
        granule = rng.choice([128, 512, 1000])
        tok = [granule * rng.randint(1, 8) for _ in range(rng.randint(2, 8))]
        return {"kind": kind, "dtype": "bf16", "dims": f"{rng.choice([4096, 5120])}x{rng.choice([4096, 12288])}",
                "ranks": _text(_ranks(rng, len(tok))), "tokens": _text(tok), "n_nano": rng.randint(2, 12),
                "granule": granule}
    if kind == "mlp":
        tok = _split(rng, _log_uniform(rng, 64, 16384), rng.randint(1, 8))
        return {"kind": kind, "dtype": "bf16", "d_model": rng.choice([1024, 2048, 4096]),
                "d_ff": rng.choice([2816, 8192, 12288]), "ranks": _text(_ranks(rng, len(tok))), "tokens": _text(tok)}
    if kind == "decoder":
        seq = rng.choice([256, 512, 777, 2048])
        tok = [seq * rng.randint(1, 4) for _ in range(rng.randint(1, 6))]
        heads, kv = rng.choice([(32, 8), (16, 4), (16, 16), (8, 1)])
        return {"kind": kind, "dtype": "bf16", "d_model": rng.choice([2048, 4096]), "d_ff": rng.choice([8192, 12288]),
                "heads": heads, "kv_heads": kv, "ranks": _text(_ranks(rng, len(tok), 128)), "tokens": _text(tok),
                "seq_len": seq}
    if kind == "attention":
        heads, kv = rng.choice([(32, 8), (16, 4), (16, 16), (8, 1)])
        return {"kind": kind, "dtype": "bf16", "heads": heads, "kv_heads": kv,
                "tokens": str(_log_uniform(rng, 512, 32768)), "seq_len": _log_uniform(rng, 100, 8192)}
    n = rng.randint(1, 16)
    return {"kind": "adamw", "dtype": rng.choice(["bf16", "f32"]), "dims": rng.choice([GATE_UP_DOWN, "4096x4096", "1000x3000"]),
            "ranks": _text(_ranks(rng, n)), "tokens": "0"}


class _Draw:
    """Seeded device tensors."""

    def __init__(self, case, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(self, *shape, std=1.0):
        t = torch.randn(*shape, device="cuda", generator=self.g, dtype=self.dtype)
        return t if std == 1.0 else t.mul_(std)

    def adapters(self, d_in, d_out, ranks):
        A = [((torch.rand(d_in, r, device="cuda", generator=self.g) * 2 - 1) / d_in ** 0.5).to(self.dtype) for r in ranks]
        B = [self.normal(r, d_out, std=0.01) for r in ranks]
        return A, B

    def projections(self, shapes, ranks):
        return {n: (self.normal(i, o, std=i ** -0.5), *self.adapters(i, o, ranks)) for n, (i, o) in shapes.items()}


def _flat(shapes, dtype=torch.float32):
    """(buffer, views): tensors of these shapes inside one zeroed buffer, each starting on a 64-element boundary --
    how a trainer holds the gradients and the optimizer state of many small adapters."""
    sizes = [(math.prod(s) + 63) // 64 * 64 for s in shapes]
    buf = torch.zeros(sum(sizes), dtype=dtype, device="cuda")
    at, views = 0, []
    for s, n in zip(shapes, sizes):
        views.append(buf[at:at + math.prod(s)].view(s))
        at += n
    return buf, views


def _flat_like(tensors, dtype):
    buf, views = _flat([t.shape for t in tensors], dtype)
    for v, t in zip(views, tensors):
        v.copy_(t)
    return buf, views


def _seq_offsets(T, seq_len):
    return list(range(0, T, seq_len)) + [T]


def prepare(case, seed):
    kind, draw_ = case["kind"], _Draw(case, seed)
    ranks, tokens = _ints(case["ranks"]) if "ranks" in case else [], _ints(case["tokens"])
    offsets, T, scales = _offsets(tokens), sum(tokens), [2.0] * len(ranks)
    st = {"kind": kind, "case": case}
    if kind in ("layer", "noalloc", "nano", "indexed"):
        st["parts"] = []
        for d_in, d_out in _dims(case):
            W, X = draw_.normal(d_in, d_out, std=0.02), draw_.normal(T, d_in)
            A, B = draw_.adapters(d_in, d_out, ranks)
            lp = tlora.LayerProblem(case["dtype"], d_in, d_out, ranks, offsets, scales, X, W, A, B)
            if kind == "noalloc":
                st["parts"].append((lp, torch.empty((T, d_out), dtype=X.dtype, device="cuda")))
                continue
            grads, views = _flat([(d_in, r) for r in ranks] + [(r, d_out) for r in ranks])
            st["parts"].append((lp, draw_.normal(T, d_out), torch.empty((T, d_out), dtype=X.dtype, device="cuda"),
                                torch.empty_like(X), views[:len(ranks)], views[len(ranks):], grads))
            if kind == "nano":
                lp._nano_ws(case["n_nano"], case["granule"])
            if kind == "indexed":
                key = torch.rand((T + case["granule"] - 1) // case["granule"], device="cuda", generator=draw_.g)
                key = key.repeat_interleave(case["granule"])[:T]
                st["index"] = torch.argsort(key, stable=True).to(torch.int32)
                n = tlora.tlora_indexed_workspace_bytes(lp.prob)
                st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return st
    if kind == "mlp":
        d, f = case["d_model"], case["d_ff"]
        layers = draw_.projections({"gate": (d, f), "up": (d, f), "down": (f, d)}, ranks)
        X, gamma = draw_.normal(T, d), torch.ones(d, device="cuda", dtype=draw_.dtype)
        st["block"] = tlora.MlpBlock(case["dtype"], d, f, ranks, offsets, scales, X, gamma, 1e-5, layers)
    elif kind == "decoder":
        d, f, h, kv = case["d_model"], case["d_ff"], case["heads"], case["kv_heads"]
        q, k = h * HEAD_DIM, kv * HEAD_DIM
        layers = draw_.projections({"q": (d, q), "k": (d, k), "v": (d, k), "o": (q, d), "gate": (d, f), "up": (d, f),
                                    "down": (f, d)}, ranks)
        X, gamma = draw_.normal(T, d), torch.ones(d, device="cuda", dtype=draw_.dtype)
        st["block"] = tlora.DecoderLayer(d, f, h, kv, 500000.0, ranks, offsets, scales, _seq_offsets(T, case["seq_len"]),
                                         X, gamma, gamma, 1e-5, layers)
    elif kind == "attention":
        h, kv = case["heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM
        st["attn"] = tlora.Attention(_seq_offsets(T, case["seq_len"]), case["heads"], case["kv_heads"], "cuda")
        Q, K, V, dO = draw_.normal(T, h), draw_.normal(T, kv), draw_.normal(T, kv), draw_.normal(T, h)
        lse = torch.empty((T, case["heads"]), dtype=torch.float32, device="cuda")
        st["tensors"] = (Q, K, V, torch.empty_like(Q), dO, lse, torch.empty_like(Q), torch.empty_like(K), torch.empty_like(V))
        return st
    elif kind == "adamw":
        params = [t for d_in, d_out in _dims(case) for ab in draw_.adapters(d_in, d_out, ranks) for t in ab]
        param, st["param"] = _flat_like(params, draw_.dtype)
        master, st["master"] = _flat_like(params, torch.float32) if case["dtype"] == "bf16" else (None, None)
        small = lambda t: torch.randn(t.shape, device="cuda", generator=draw_.g) * 1e-3
        _, st["grad"] = _flat_like([small(t) for t in params], torch.float32)
        m, st["m"] = _flat_like([small(t) for t in params], torch.float32)
        v, st["v"] = _flat_like([small(t) ** 2 for t in params], torch.float32)
        st["out"] = [t for t in (param, master, m, v) if t is not None]
        n = tlora.tlora_adamw_workspace_bytes(len(params))
        st["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return st
    st["dOut"], st["Out"], st["dX"] = draw_.normal(T, d), torch.empty_like(X), torch.empty_like(X)
    names = list(layers)
    shapes = [t.shape for n in names for ab in layers[n][1:] for t in ab]
    st["flat"], views = _flat(shapes)
    it = iter(views)
    st["grads"] = {n: tuple([next(it) for _ in ranks] for _ in range(2)) for n in names}
    return st


def run(st):
    kind, case = st["kind"], st["case"]
    stream = int(torch.cuda.current_stream().cuda_stream)
    if kind == "noalloc":
        lp, Y = st["parts"][0]
        tlora.tlora_fwd_noalloc(lp.prob, Y.data_ptr(), stream)
        return Y
    if kind == "layer":
        for lp, dY, Y, dX, dA, dB, _ in st["parts"]:
            lp.fwd(Y)
            lp.bwd(dY, dX, dA, dB, reuse_S=True)
        return [[Y, dX, grads] for _, _, Y, dX, _, _, grads in st["parts"]]
    if kind == "nano":
        lp, dY, Y, dX, dA, dB, grads = st["parts"][0]
        lp.fwd_nano(case["n_nano"], case["granule"], Y)
        lp.bwd_nano(case["n_nano"], case["granule"], dY, dX, dA, dB)
        return [Y, dX, grads]
    if kind == "indexed":
        lp, dY, Y, dX, dA, dB, grads = st["parts"][0]
        ws, index = st["ws"], st["index"]
        tlora.tlora_fwd_indexed(lp.prob, index.data_ptr(), Y.data_ptr(), ws.data_ptr(), ws.numel(), stream)
        tlora.tlora_bwd_indexed(lp.prob, index.data_ptr(), dY.data_ptr(), dX.data_ptr(), [t.data_ptr() for t in dA],
                                [t.data_ptr() for t in dB], tlora.TLORA_BWD_REUSE_S, ws.data_ptr(), ws.numel(), stream)
        return [Y, dX, grads]
    if kind == "attention":
        Q, K, V, O, dO, lse, dQ, dK, dV = st["tensors"]
        st["attn"].fwd(Q, K, V, O, lse)
        st["attn"].bwd(Q, K, V, O, dO, lse, dQ, dK, dV)
        return [O, lse, dQ, dK, dV]
    if kind == "adamw":
        master = st["master"] or [None] * len(st["param"])
        tens = [dict(param=p.data_ptr(), master=w.data_ptr() if w is not None else 0, grad=g.data_ptr(), m=m.data_ptr(),
                     v=v.data_ptr(), n=p.numel(), lr=1e-4, weight_decay=0.01, step=10)
                for p, w, g, m, v in zip(st["param"], master, st["grad"], st["m"], st["v"])]
        tlora.tlora_adamw_step(tens, tlora.TLORA_BF16 if case["dtype"] == "bf16" else tlora.TLORA_F32,
                               st["ws"].data_ptr(), st["ws"].numel(), stream)
        return st["out"]
    st["block"].fwd(st["Out"])
    st["block"].bwd(st["dOut"], st["dX"], st["grads"])
    return [st["Out"], st["dX"], st["flat"]]


def _projection_work(dims, ranks, tokens, elt, backward=True):
    """Weights and adapters read, adapter gradients written; products of the backbone and of the rank side."""
    T, tr, R = sum(tokens), sum(t * r for t, r in zip(tokens, ranks)), sum(ranks)
    flops = nbytes = 0
    for d_in, d_out in dims:
        flops += (4 if backward else 2) * T * d_in * d_out + (6 if backward else 2) * (d_in + d_out) * tr
        nbytes += elt * (d_in * d_out + R * (d_in + d_out)) + (4 * R * (d_in + d_out) if backward else 0)
    return flops, nbytes


def _attention_pairs(T, seq_len, heads):
    full, rest = divmod(T, seq_len)
    return heads * (full * seq_len * (seq_len + 1) // 2 + rest * (rest + 1) // 2)


def work(case):
    kind, elt = case["kind"], 2 if case["dtype"] == "bf16" else 4
    ranks, tokens = _ints(case["ranks"]) if "ranks" in case else [], _ints(case["tokens"])
    T = sum(tokens)
    if kind in ("layer", "nano", "indexed", "noalloc"):
        bwd = kind != "noalloc"
        flops, nbytes = _projection_work(_dims(case), ranks, tokens, elt, bwd)
        # X and dY in, Y and dX out
        nbytes += sum((2 if bwd else 1) * elt * T * (i + o) for i, o in _dims(case)) + (4 * T if kind == "indexed" else 0)
    elif kind == "mlp":
        d, f = case["d_model"], case["d_ff"]
        flops, nbytes = _projection_work([(d, f), (d, f), (f, d)], ranks, tokens, elt)
        nbytes += 4 * elt * T * d
    elif kind == "decoder":
        d, f = case["d_model"], case["d_ff"]
        q, k = case["heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM
        flops, nbytes = _projection_work([(d, q), (d, k), (d, k), (q, d), (d, f), (d, f), (f, d)], ranks, tokens, elt)
        flops += 14 * _attention_pairs(T, case["seq_len"], case["heads"]) * HEAD_DIM
        nbytes += 4 * elt * T * d
    elif kind == "attention":
        h, kv = case["heads"] * HEAD_DIM, case["kv_heads"] * HEAD_DIM
        flops = 14 * _attention_pairs(T, case["seq_len"], case["heads"]) * HEAD_DIM
        # Q, dO in, O, dQ out; K, V in, dK, dV out; lse out
        nbytes = 4 * elt * T * (h + kv) + 4 * T * case["heads"]
    else:
        n = sum(ranks) * sum(i + o for i, o in _dims(case))
        # grad, m, v and the fp32 weights in; m, v and the weights out; the bf16 copy out
        flops, nbytes = 15 * n, (30 if case["dtype"] == "bf16" else 28) * n
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the error measured against float64 references of the same inputs: bf16 layers 1.7e-3 (one
    rounding of Y / dX), attention 2.5e-3 (bf16 probabilities and score gradients), the MLP block 4.1e-3 and the decoder
    layer 7.2e-3 (chains of bf16 tensors), fp32 layers 3.9e-8 (64-bit sums), optimizer 7e-8 on fp32 state (its bf16 copy: a
    few roundings that fall on the other side)."""
    if case["kind"] == "adamw":
        return {"rel": 4e-5 if case["dtype"] == "bf16" else 4e-7}
    if case["dtype"] == "f32":
        return {"rel": 2e-7}
    return {"rel": {"mlp": 1.6e-2, "decoder": 2.8e-2, "attention": 1e-2}.get(case["kind"], 7e-3)}
