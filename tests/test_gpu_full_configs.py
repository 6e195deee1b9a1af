"""GPU parity at the benchmark's full sizes and launch configuration.

The oracle is O(n^2) per channel, so at full size it runs on a sample of head-tensors (whole
head-tensors, all rows and channels, on several host threads) that always includes the first and
last layer and K head-tensors with outlier channels; everything else is covered by properties
that hold at any size (sinks untouched, nothing written past the retained rows).
"""
import math
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth
from paper_2505_00570_amd.cache import CompressedKVCache
from oracle import freqkv_oracle as orc

from _util import TOL_BF16, bf16_round, bf16_ulp, f64, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda"
THREADS = min(16, os.cpu_count() or 1)


def _say(msg):
    print(msg, flush=True)


def _sample_heads(wl, count, seed):
    """(kv, layer, batch, head) tuples: first/last layer always in, rest seeded-random."""
    rng = np.random.default_rng(seed)
    picks = {(0, 0, 0, 0), (1, wl.n_layers - 1, wl.batch - 1, wl.n_heads - 1), (0, wl.n_layers - 1, 0, 0)}
    while len(picks) < count:
        picks.add((int(rng.integers(2)), int(rng.integers(wl.n_layers)), int(rng.integers(wl.batch)),
                   int(rng.integers(wl.n_heads))))
    return sorted(picks)


def _check_sample(wl, before, after, tap, p, picks, tol=TOL_BF16, n_cols=None):
    """before/after: dict (kv,l,b,h) -> host tensors [W, d]; tap: dict -> [Lc, d] fp32 or None.
    n_cols: compare only that many seeded channels of each sampled head-tensor (all when None)."""
    S, W, lc = wl.n_sink, wl.window, p.retained_len

    def one(key):
        cols = slice(None)
        if n_cols is not None:
            cols = np.sort(np.random.default_rng(hash(key) & 0xffff).choice(wl.head_dim, n_cols, replace=False))
        x = np.ascontiguousarray(f64(before[key])[:, cols])
        ref = orc.compress_head(x, W, W, S, wl.retain_ratio)[S:]
        got = f64(after[key][S:S + lc])[:, cols]
        rms = math.sqrt(float((ref ** 2).mean()))
        store = float((np.abs(got - ref) - 0.5 * bf16_ulp(ref)).max()) / rms
        raw = float(np.abs(got - ref).max()) / rms
        floor = float(np.abs(bf16_round(ref) - ref).max()) / rms
        t = None
        if tap is not None:
            yt = f64(tap[key])[:, cols]
            t = rel_err(yt, ref)
            assert np.array_equal(got, bf16_round(yt)), key
        assert torch.equal(after[key][:S], before[key][:S]), key
        return store, raw, floor, t

    with ThreadPoolExecutor(max_workers=THREADS) as ex:
        res = list(ex.map(one, picks))
    worst_store = max(r[0] for r in res)
    worst_raw = max(r[1] for r in res)
    worst_floor = max(r[2] for r in res)
    worst_tap = max((r[3] for r in res if r[3] is not None), default=None)
    _say(f"  {len(picks)} head-tensors: fp32-tap err/rms {worst_tap}, stored-bf16 err/rms raw {worst_raw:.3e} "
         f"(bf16 grid floor of the oracle itself {worst_floor:.3e}), beyond the grid {worst_store:.3e}")
    if worst_tap is not None:
        assert worst_tap <= tol
    assert worst_store <= tol
    return worst_raw, worst_floor


def _one_trigger_full(wl, n_pick, seed, with_tap, extra_picks=(), expect=None, flags=0, variant=None):
    k, v = synth.empty_cache(wl, DEV)
    synth.KVSource(wl, seed, DEV).fill(k, v, 0, wl.window)
    L = binding.layout_for(k, flags=flags)
    _, p = fk.plan(L, wl.n_heads, wl.head_dim, wl.window, wl.window, wl.n_sink, wl.retain_ratio)
    if variant is not None:
        assert p.variant == variant and p.runs == (variant if flags else 7)
    if expect is not None:
        assert (p.span_len, p.retained_len, p.head_tensors) == expect
    ws = torch.empty(max(p.workspace_bytes, 256), dtype=torch.uint8, device=DEV)
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    tapt = None
    if with_tap:
        tapt = torch.empty(2, wl.n_layers, wl.batch, wl.n_heads, p.retained_len, wl.head_dim,
                           dtype=torch.float32, device=DEV)
        L.tap_f32 = tapt.data_ptr()
    picks = sorted(set(_sample_heads(wl, n_pick, seed)) | set(extra_picks))
    src = (k, v)
    before = {key: src[key[0]][key[1], key[2], key[3]].cpu().clone() for key in picks}
    sinks_k = k[:, :, :, :wl.n_sink].clone()
    sinks_v = v[:, :, :, :wl.n_sink].clone()
    assert fk.compress(k, v, L, wl.n_heads, wl.head_dim, wl.window, wl.window, wl.n_sink, wl.retain_ratio) == 0
    torch.cuda.synchronize()
    after = {key: src[key[0]][key[1], key[2], key[3]].cpu() for key in picks}
    tap = {key: tapt[key].cpu() for key in picks} if with_tap else None
    # properties over the WHOLE cache: sinks bit-identical, retained rows finite
    assert torch.equal(k[:, :, :, :wl.n_sink], sinks_k) and torch.equal(v[:, :, :, :wl.n_sink], sinks_v)
    assert torch.isfinite(k[:, :, :, :p.new_len].float()).all()
    assert torch.isfinite(v[:, :, :, :p.new_len].float()).all()
    return _check_sample(wl, before, after, tap, p, picks)


def test_llama2_7b_one_layer_full():
    """Config 2: 32 heads x 4096 x 128, every one of the 64 head-tensors against the oracle."""
    wl = synth.WORKLOADS["llama2_7b_layer"]
    _say(f"config 2 {wl.name}")
    k, v = synth.empty_cache(wl, DEV)
    synth.KVSource(wl, 0, DEV).fill(k, v, 0, wl.window)
    L = binding.layout_for(k)
    _, p = fk.plan(L, wl.n_heads, wl.head_dim, wl.window, wl.window, wl.n_sink, wl.retain_ratio)
    assert (p.span_len, p.retained_len, p.head_tensors, p.variant) == (4092, 2046, 64, 6)
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device=DEV)
    tapt = torch.empty(2, 1, 1, 32, p.retained_len, 128, dtype=torch.float32, device=DEV)
    L.workspace, L.workspace_bytes, L.tap_f32 = ws.data_ptr(), p.workspace_bytes, tapt.data_ptr()
    picks = [(kv, 0, 0, h) for kv in range(2) for h in range(32)]
    src = (k, v)
    before = {key: src[key[0]][0, 0, key[3]].cpu().clone() for key in picks}
    assert fk.compress(k, v, L, 32, 128, 4096, 4096, 4, 0.5) == 0
    torch.cuda.synchronize()
    after = {key: src[key[0]][0, 0, key[3]].cpu() for key in picks}
    tap = {key: tapt[key].cpu() for key in picks}
    _check_sample(wl, before, after, tap, p, picks)


# the full-size triggers run twice: the near/far form (the default, though the plan's variant is the factored transform) and
# the matrix form
FORMS = [pytest.param(0, 6, id="nearfar"), pytest.param(binding.FLAG_DENSE, 5, id="matrix")]


@pytest.mark.parametrize("flags,variant", FORMS)
def test_llama3_8b_gqa_full_size_trigger(flags, variant):
    """Config 4 at full size (the launch configuration bench.py times): 512 head-tensors, span 8188."""
    wl = synth.WORKLOADS["llama3_8b_128k"]
    _say(f"config 4 {wl.name} (one full-size trigger, variant {variant})")
    _one_trigger_full(wl, n_pick=16, seed=4, with_tap=True, flags=flags, variant=variant)


@pytest.mark.parametrize("flags,variant", FORMS)
def test_llama2_7b_full_model_trigger(flags, variant):
    """Config 3 at full size: 32 layers x 32 heads, 2048 head-tensors, span 4092."""
    wl = synth.WORKLOADS["llama2_7b_32k"]
    _say(f"config 3 {wl.name} (one full-size trigger, variant {variant})")
    _one_trigger_full(wl, n_pick=32, seed=3, with_tap=False, flags=flags, variant=variant)


@pytest.mark.parametrize("flags,variant", FORMS)
def test_decode_b8_full_size_trigger(flags, variant):
    """Config 5 at full size (the launch `bench.py --workload decode_b8_256k` times): batch 8 x 32 layers x
    32 heads = 16384 head-tensors of span 4092 in one call, 17.2 GB of cache and 8.6 GB of workspace.
    20 whole head-tensors against the oracle (first and last layer, first and last sequence of the
    batch, K heads with their outlier channels), sinks of the whole cache bit for bit."""
    wl = synth.WORKLOADS["decode_b8_256k"]
    _say(f"config 5 {wl.name} (one full-size trigger, variant {variant})")
    extra = [(0, wl.n_layers - 1, wl.batch - 1, 5), (0, 0, wl.batch - 1, wl.n_heads - 1), (1, 0, 0, 0),
             (0, 17, 3, 11)]
    _one_trigger_full(wl, n_pick=16, seed=5, with_tap=False, extra_picks=extra, expect=(4092, 2046, 16384),
                      flags=flags, variant=variant)


def _iterative(wl, seed, picks_per_trigger, max_triggers=None, n_cols=None):
    """Stream wl.total_tokens through the cache; teacher-forced parity on sampled head-tensors at
    every trigger (the oracle starts from the bits the GPU holds just before that trigger)."""
    W, S = wl.window, wl.n_sink
    cache = CompressedKVCache(wl.n_layers, wl.batch, wl.n_heads, wl.head_dim, W, S, wl.retain_ratio, wl.dtype, DEV)
    src = synth.KVSource(wl, seed, DEV)
    free = cache.free_after_trigger
    fed, worst = 0, 0.0
    while fed < wl.total_tokens:
        if cache.cur_len >= W:
            if max_triggers is not None and cache.triggers >= max_triggers:
                break
            picks = _sample_heads(wl, picks_per_trigger, seed * 1000 + cache.triggers)
            kv = (cache.k, cache.v)
            before = {key: kv[key[0]][key[1], key[2], key[3]].cpu().clone() for key in picks}
            assert cache.compress() == 0
            torch.cuda.synchronize()
            after = {key: kv[key[0]][key[1], key[2], key[3]].cpu() for key in picks}
            raw, _ = _check_sample(wl, before, after, None, cache.plan, picks, n_cols=n_cols)
            worst = max(worst, raw)
        take = min(wl.total_tokens - fed, W - cache.cur_len)
        assert take == (W if fed == 0 else min(free, wl.total_tokens - fed))
        kn = torch.empty(wl.n_layers, wl.batch, wl.n_heads, take, wl.head_dim, dtype=wl.dtype, device=DEV)
        vn = torch.empty_like(kn)
        src.fill(kn, vn, 0, take)
        cache.append(kn, vn)
        fed += take
    return cache, worst


def test_llama2_7b_32k_iterative_prefill():
    """Config 3 schedule: 32K tokens, window 4096 -> 15 triggers (first after 4096 tokens, then every 2046).
    Eight layers of the model keep the run short; the per-trigger launch is the same kernel."""
    wl = synth.small(synth.WORKLOADS["llama2_7b_32k"], n_layers=8)
    _say("config 3 schedule: 32K tokens, 8 layers x 32 heads")
    cache, worst = _iterative(wl, seed=33, picks_per_trigger=8)
    assert cache.triggers == 15 == orc.trigger_count(32768, 4096, 4, 0.5)
    _say(f"  15 triggers, worst raw stored err/rms {worst:.3e}")


def test_llama3_8b_128k_iterative_prefill():
    """Config 4 schedule: 128K tokens, window 8192 -> 31 triggers; 4 layers x 8 KV heads."""
    wl = synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=4)
    _say("config 4 schedule: 128K tokens, 4 layers x 8 KV heads")
    cache, worst = _iterative(wl, seed=44, picks_per_trigger=8, n_cols=16)
    assert cache.triggers == 31 == orc.trigger_count(131072, 8192, 4, 0.5)
    _say(f"  31 triggers, worst raw stored err/rms {worst:.3e}")


def test_decode_batch8_stream():
    """Config 5 shape (batch 8, 32 heads, window 4096) on 2 layers; the first 12 triggers of the
    256K-token stream (each refill stands for 2046 decode steps)."""
    wl = synth.small(synth.WORKLOADS["decode_b8_256k"], n_layers=2)
    _say("config 5: batch 8 x 32 heads, 2 layers, 12 triggers")
    cache, worst = _iterative(wl, seed=55, picks_per_trigger=6, max_triggers=12)
    assert cache.triggers == 12
    assert orc.trigger_count(262144, 4096, 4, 0.5) == 127
    _say(f"  worst raw stored err/rms {worst:.3e}")


# ------------------------------------------------------------------------------------------
# free-running drift over the whole schedules: two head-tensors carried in fp64 on the host
# ------------------------------------------------------------------------------------------

def _free_running(wl, seed, n_cols=16):
    """Stream wl.total_tokens through the cache.  Two head-tensors (a K head with its outlier channels, a V
    head of the last layer) are carried on the host in fp64 through EVERY trigger without ever seeing the
    GPU's rows again (free running), on n_cols channels.  The operator has spectral norm sqrt(Lc/n) < 1
    (it keeps Lc of n orthonormal directions and rescales), so with r_T the teacher-forced error of trigger T
    (GPU result minus the oracle on the GPU's own pre-trigger bits) the drift D_T = GPU - free-running obeys
    ||D_T|| <= sqrt(Lc/n) ||D_{T-1}|| + ||r_T||  (Frobenius norm over the retained block): asserted at every
    trigger.  Returns (triggers, worst max-abs drift / RMS, last bound / norm of the block)."""
    W, S = wl.window, wl.n_sink
    cache = CompressedKVCache(wl.n_layers, wl.batch, wl.n_heads, wl.head_dim, W, S, wl.retain_ratio, wl.dtype, DEV)
    src = synth.KVSource(wl, seed, DEV)
    lc = cache.plan.retained_len
    gain = math.sqrt(lc / (W - S))
    picks = [(0, 0, 0, 0), (1, wl.n_layers - 1, wl.batch - 1, wl.n_heads - 1)]
    cols, free, bound = {}, {}, {key: 0.0 for key in picks}
    fed, worst_rel, last = 0, 0.0, 0.0
    while fed < wl.total_tokens:
        kv = (cache.k, cache.v)
        if cache.cur_len >= W:
            before = {key: f64(kv[key[0]][key[1], key[2], key[3], :W])[:, cols[key]] for key in picks}
            assert cache.compress() == 0
            torch.cuda.synchronize()
            for key in picks:
                got = f64(kv[key[0]][key[1], key[2], key[3], S:S + lc])[:, cols[key]]
                teacher = orc.compress_head(before[key], W, W, S, wl.retain_ratio)[S:]
                free[key] = orc.compress_head(free[key], W, W, S, wl.retain_ratio)
                r = float(np.linalg.norm(got - teacher))
                drift = got - free[key][S:]
                bound[key] = gain * bound[key] + r
                dn = float(np.linalg.norm(drift))
                assert dn <= bound[key] * (1 + 1e-9) + 1e-9, (key, cache.triggers, dn, bound[key])
                rms = math.sqrt(float((free[key][S:] ** 2).mean()))
                rel = float(np.abs(drift).max()) / rms
                # element-wise: every trigger adds at most the tolerance plus half a bf16 step of the largest
                # retained value, and earlier errors shrink by sqrt(Lc/n) per trigger (a geometric series)
                floor = 0.5 * float(bf16_ulp(np.abs(free[key][S:]).max())) / rms
                assert rel <= (TOL_BF16 + floor) / (1.0 - gain), (key, cache.triggers, rel, floor)
                worst_rel = max(worst_rel, rel)
                last = bound[key] / float(np.linalg.norm(free[key][S:]))
        take = min(wl.total_tokens - fed, W - cache.cur_len)
        kn = torch.empty(wl.n_layers, wl.batch, wl.n_heads, take, wl.head_dim, dtype=wl.dtype, device=DEV)
        vn = torch.empty_like(kn)
        src.fill(kn, vn, 0, take)
        new = (kn, vn)
        for key in picks:
            rows = f64(new[key[0]][key[1], key[2], key[3]])
            if key not in cols:
                # the channels with the largest RMS first (K: the outlier channels), then seeded others
                order = np.argsort(-np.sqrt((rows ** 2).mean(axis=0)))
                rest = np.random.default_rng(seed).permutation(order[4:])[:n_cols - 4]
                cols[key] = np.sort(np.concatenate([order[:4], rest]))
                free[key] = np.empty((0, n_cols))
            free[key] = np.concatenate([free[key], rows[:, cols[key]]], axis=0)
        cache.append(kn, vn)
        fed += take
    return cache.triggers, worst_rel, last


@pytest.mark.parametrize("name,layers,d,count", [("llama2_7b_32k", 2, 128, 15), ("llama3_8b_128k", 2, 128, 31),
                                                 ("decode_b8_256k", 1, 128, 127), ("llama2_7b_32k", 2, 80, 15)])
def test_free_running_drift_over_the_whole_schedule(name, layers, d, count):
    """Configs 3, 4, 5: all 15 / 31 / 127 triggers of the schedule, two head-tensors free running in fp64; once with a head size
    that takes the factored transform."""
    wl = synth.small(synth.WORKLOADS[name], n_layers=layers, head_dim=d)
    triggers, worst, bound_rel = _free_running(wl, seed=90 + count)
    assert triggers == count == orc.trigger_count(wl.total_tokens, wl.window, wl.n_sink, wl.retain_ratio)
    _say(f"free running {name}: {triggers} triggers, worst max-abs drift / RMS {worst:.3e}; "
         f"||drift|| bound from the teacher-forced errors and the gain sqrt(Lc/n): {bound_rel:.3e} of the block norm")
