"""Performance cases of the library: what a FreqKV serving or prefilling program has it do, call by call.

Every case goes through the public binding with buffers, layout and workspace laid out once, as a program that
keeps a compressed KV cache holds them.  Shapes are those of the benchmark configurations (synth.WORKLOADS), of
the tests, or generic.  Five kinds of call:

  compress   one trigger over all layers' K and V of a full cache
  ragged     a trigger for a batch whose sequences hold different numbers of tokens
  decode     attention of one new token per sequence over the cached rows (one layer, as a decoder calls it
             between its projections, or all layers of a cache in one call)
  decode_ragged   the same for a batch of sequences of different lengths
  prefill    attention of an incoming chunk over the cached rows
"""
import math

import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding

BF16_BYTES, F32_BYTES = 2, 4


def _case(kind, name=None, **kw):
    c = dict(kind=kind, dtype="bf16", layers=1, batch=1, kv_heads=8, q_heads=32, d=128)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def _trigger(name=None, kind="compress", window=8192, sinks=4, ratio=0.5, tail=0, **kw):
    return _case(kind, name, window=window, sinks=sinks, ratio=ratio, tail=tail, **kw)


def listed():
    return [
        # the smallest benchmark configuration: one fp32 head, window 512; a call is launch and latency
        _trigger("compress_tiny_f32", window=512, dtype="f32", kv_heads=1, d=64),
        # one LLaMA-2-7B layer: a decoder that triggers layer by layer
        _trigger("compress_layer_4k", window=4096, kv_heads=32),
        # the benchmark's headline: a whole LLaMA-3-8B cache during a 128K prefill
        _trigger("compress_llama3_8k", window=8192, layers=32),
        # the largest configuration: batch-8 decoding of LLaMA-2-7B, 17 GB of cache
        _trigger("compress_llama2_b8_4k", window=4096, layers=32, batch=8, kv_heads=32),
        # another retention ratio on the LLaMA-3-8B cache
        _trigger("compress_llama3_quarter", window=8192, layers=32, ratio=0.25),
        # a window and a sink count off the paper's defaults, and a tail of newer tokens behind the window
        _trigger("compress_window_6100", window=6100, sinks=17, layers=8, tail=37),
        # a serving batch: every sequence compacts on its own schedule
        _trigger("compress_ragged_b6", kind="ragged", window=4096, layers=16, batch=6, lens_seed=3),
        # one layer of one sequence per generated token: the smallest and by far the most frequent call
        _case("decode", "decode_layer_b1", cur_len=6147),
        # all layers of a full LLaMA-3-8B cache in one call
        _case("decode", "decode_llama3_all_layers", layers=32, cur_len=8192),
        # a serving batch of sequences at different points of their windows, one layer
        _case("decode_ragged", "decode_ragged_b16", batch=16, cur_len=8192, lens_seed=5),
        # prefill: the 4094 tokens that fit behind 4098 compacted rows, one layer
        _case("prefill", "prefill_layer_chunk", cur_len=8192, q_len=4094),
        # a short turn of a conversation behind an already filled cache, one layer
        _case("prefill", "prefill_short_turn", cur_len=5001, q_len=301),
    ]


# ---------------------------------------------------------------- drawn cases

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fit(c, rows, most):
    """Fewer layers, then fewer sequences, until the K and V rows of the case take at most `most` bytes."""
    elem = F32_BYTES if c["dtype"] == "f32" else BF16_BYTES

    def size():
        return 2 * c["layers"] * c["batch"] * c["kv_heads"] * rows * c["d"] * elem

    while size() > most and c["layers"] > 1:
        c["layers"] = max(1, c["layers"] // 2)
    while size() > most and c["batch"] > 1:
        c["batch"] = max(1, c["batch"] // 2)
    return c


def draw(rng):
    kind = rng.choice(["compress", "compress", "compress", "ragged", "decode", "decode", "decode_ragged",
                       "prefill", "prefill"])
    heads = rng.choice([1, 2, 4, 8, 8, 8, 16, 32])
    d = rng.choice([64, 128, 128, 128])
    if kind in ("compress", "ragged"):
        # the paper's kind of window (a power of two with 4 sinks) more often than an arbitrary one
        usual = rng.random() < 0.55
        window = rng.choice([1024, 2048, 4096, 8192]) if usual else _log_int(rng, 200, 16384)
        sinks = 4 if usual else rng.choice([0, 1, 4, 8, 16, 64])
        ratio = 0.5 if rng.random() < 0.7 else rng.choice([0.25, 0.375, 0.6, 0.75, 0.9])
        c = _trigger(kind=kind, window=window, sinks=sinks, ratio=ratio, kv_heads=heads, d=d,
                     layers=_log_int(rng, 1, 40), batch=_log_int(rng, 1, 8),
                     tail=rng.choice([0, 0, 0, rng.randint(1, 300)]))
        if kind == "ragged":
            c["batch"], c["lens_seed"] = rng.randint(2, 12), rng.randint(0, 1 << 20)
        elif rng.random() < 0.12:                          # small fp32 caches, as the tests and the first configuration use
            c.update(dtype="f32", window=_log_int(rng, 200, 2048), sinks=4, kv_heads=min(heads, 8), layers=rng.randint(1, 4), batch=1)
        return _fit(c, c["window"] + c["tail"], 4 << 30)
    group = rng.choice([1, 2, 4, 4, 4, 8])
    if kind == "prefill":
        cur = _log_int(rng, 256, 8192)
        c = _case(kind, layers=rng.choice([1, 1, 1, 2, 4]), batch=rng.choice([1, 1, 1, 2, 4]), kv_heads=heads,
                  q_heads=min(32, heads * group) // heads * heads, cur_len=cur,
                  q_len=rng.choice([_log_int(rng, 2, cur), _log_int(rng, 16, min(cur, 1024)), max(1, cur // 2), cur]))
        while c["layers"] * c["batch"] * c["q_heads"] * c["q_len"] > 32 * 4 * 8192 and c["layers"] * c["batch"] > 1:
            c["layers"], c["batch"] = max(1, c["layers"] // 2), max(1, c["batch"] // 2)
        return c
    c = _case(kind, dtype="f32" if rng.random() < 0.1 else "bf16", layers=rng.choice([1, 1, 1, 1, 8, 32]),
              batch=_log_int(rng, 1, 64), kv_heads=heads, q_heads=heads * group,
              d=rng.choice([64, 128, 128, 128, 128, 256]), cur_len=_log_int(rng, 64, 16384))
    if kind == "decode_ragged":
        c["batch"], c["lens_seed"] = max(2, c["batch"]), rng.randint(0, 1 << 20)
    return _fit(c, c["cur_len"], 4 << 30)


# ---------------------------------------------------------------- the calls

def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _lens(case):
    """Tokens held by the sequences of a ragged batch (host integers, fixed by the case)."""
    import random
    r = random.Random(case["lens_seed"])
    if case["kind"] == "ragged":
        # most sequences have just reached the window, some run a little behind or ahead of it
        w = case["window"]
        return [r.choice([w, w, w + r.randint(1, 48), r.randint(w // 2, w - 1)]) for _ in range(case["batch"])]
    return [r.randint(max(1, case["cur_len"] // 2), case["cur_len"]) for _ in range(case["batch"])]


def _rows(case):
    if case["kind"] == "compress":
        return case["window"] + case["tail"]
    if case["kind"] == "ragged":
        return case["window"] + 48
    return case["cur_len"]


def _states(case, gen, rho, outliers):
    """[layer, batch, head, token, dim] states, correlated along the tokens as cached keys and values are
    (autoregressive, low-frequency dominated); keys have a few outlier channels per head."""
    shape = (case["batch"], case["kv_heads"], _rows(case), case["d"])
    out = torch.empty((case["layers"],) + shape, dtype=_dtype(case), device="cuda")
    for layer in range(case["layers"]):
        for b in range(case["batch"]):
            x = torch.randn(shape[1:], generator=gen, device="cuda")
            step = 1
            while step < 32 and step < shape[2]:            # x_t + rho x_{t-1} + rho^2 x_{t-2} + ...
                y = x.clone()
                y[:, step:].add_(x[:, :-step], alpha=rho ** step)
                x, step = y, 2 * step
            if outliers:
                scale = torch.ones((shape[1], 1, shape[3]), device="cuda")
                idx = torch.rand((shape[1], 1, shape[3]), generator=gen, device="cuda").topk(4, dim=2).indices
                x.mul_(scale.scatter_(2, idx, 8.0))
            out[layer, b] = x.to(out.dtype)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    k = _states(case, gen, 0.9, True)
    v = _states(case, gen, 0.8, False)
    L = binding.layout_for(k)
    s = dict(case=case, k=k, v=v, layout=L, stream=torch.cuda.current_stream())
    hkv, d, kind = case["kv_heads"], case["d"], case["kind"]
    if kind in ("compress", "ragged"):
        cur = case["window"] + case["tail"] if kind == "compress" else case["window"]
        _, p = fk.plan(L, hkv, d, cur, case["window"], case["sinks"], case["ratio"])
        need = p.workspace_bytes
        if kind == "compress":
            s["result"] = [k[:, :, :, :p.new_len], v[:, :, :, :p.new_len]]
        else:
            s["cur_lens"] = _lens(case)
            after = [p.new_len + t - case["window"] if t >= case["window"] else t for t in s["cur_lens"]]
            s["result"] = [x[:, b, :, :n] for b, n in enumerate(after) for x in (k, v)]
    else:
        hq, dt = case["q_heads"], _dtype(case)
        n_q = (case["q_len"],) if kind == "prefill" else ()
        q = torch.randn((case["layers"], case["batch"], hq) + n_q + (d,), generator=gen, device="cuda") * 0.5
        s["q"] = q.to(dt)
        s["out"] = torch.empty_like(s["q"])
        if kind == "prefill":
            _, p = fk.attend_prefill_plan(L, hq, hkv, d, case["cur_len"], case["q_len"])
        else:
            _, p = fk.attend_plan(L, hq, hkv, d, case["cur_len"])
        need = p.workspace_bytes
        if kind == "decode_ragged":
            s["cur_lens"] = torch.tensor(_lens(case), dtype=torch.int32, device="cuda")
    s["workspace"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = s["workspace"].data_ptr(), s["workspace"].numel()
    return s


ROPE_BASE = 500000.0


def run(s):
    c, k, v, L = s["case"], s["k"], s["v"], s["layout"]
    kind = c["kind"]
    if kind == "compress":
        fk.compress(k, v, L, c["kv_heads"], c["d"], c["window"] + c["tail"], c["window"], c["sinks"], c["ratio"],
                    s["stream"])
        return s["result"]                                  # the rows the caches hold after the call
    if kind == "ragged":
        fk.compress_ragged(k, v, L, c["kv_heads"], c["d"], s["cur_lens"], c["window"], c["sinks"], c["ratio"],
                           s["stream"])
        return s["result"]
    if kind == "decode":
        fk.attend_decode(s["q"], k, v, s["out"], None, L, c["q_heads"], c["kv_heads"], c["d"], c["cur_len"], -1,
                         ROPE_BASE, s["stream"])
    elif kind == "decode_ragged":
        fk.attend_decode_ragged(s["q"], k, v, s["out"], None, L, c["q_heads"], c["kv_heads"], c["d"], s["cur_lens"],
                                c["cur_len"], ROPE_BASE, s["stream"])
    else:
        fk.attend_prefill(s["q"], k, v, s["out"], None, L, c["q_heads"], c["kv_heads"], c["d"], c["cur_len"],
                          c["q_len"], ROPE_BASE, s["stream"])
    return s["out"]


# ---------------------------------------------------------------- what a pass cannot do without

def _retained(case):
    n = case["window"] - case["sinks"]
    return n, min(n, max(1, int(case["ratio"] * n + 1e-9)))


def work(case):
    e = F32_BYTES if case["dtype"] == "f32" else BF16_BYTES
    d, hkv, kind = case["d"], case["kv_heads"], case["kind"]
    if kind in ("compress", "ragged"):
        n, lc = _retained(case)
        lens = [case["window"] + case["tail"]] * case["batch"] if kind == "compress" else _lens(case)
        due = [t for t in lens if t >= case["window"]]
        columns = 2 * case["layers"] * hkv * d
        # span read once, retained rows written once, tail moved; a fast transform of each length
        rows = sum(n + lc + 2 * (t - case["window"]) for t in due)
        fast = 2.5 * (n * math.log2(n) + lc * math.log2(max(lc, 2)))
        return {"bytes": float(columns * rows * e), "flops": float(columns * fast * len(due))}
    units, hq = case["layers"], case["q_heads"]
    if kind == "prefill":
        q, cur = case["q_len"], case["cur_len"]
        seen = q * (cur - q) + q * (q + 1) / 2
        return {"bytes": float(units * case["batch"] * (2 * hkv * cur + 2 * hq * q) * d * e),
                "flops": float(4.0 * units * case["batch"] * hq * seen * d)}
    lens = [case["cur_len"]] * case["batch"] if kind == "decode" else _lens(case)
    return {"bytes": float(units * sum(2 * hkv * t + 2 * hq for t in lens) * d * e),
            "flops": float(4.0 * units * hq * sum(lens) * d)}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}
    # bf16 caches: one rounding of the result to bf16 and fp16 or bf16 operands on the matrix cores
    return {"rel": 1e-2, "max": 0.1}
