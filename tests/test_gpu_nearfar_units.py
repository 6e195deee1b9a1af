"""GPU parity of the near/far form by units (spans of 2 or 4 times the retained length) against the fp64 CPU oracle, every element:
the shortest and longest spans that it takes and their neighbours that it leaves, last leaves with 48 to 64 rows, incomplete groups
and blocks, spans that fit the ring, that turn round in it, and with held blocks; more tasks than workgroups; token-major strides."""
import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from oracle import freqkv_oracle as orc

from _util import TOL_BF16, f64
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

SPANS = [
    # ratio 1/2: 1000 and 1008 rows leave 24 and 16 rows of the last unit beyond the span (the first of them is refused); 9 units;
    # 11, 12 and 13 units around the ring; 33 units; the longest that leaves nine ring slots, and the next
    (1000, 0.5), (1008, 0.5), (1024, 0.5), (1150, 0.5), (1404, 0.5), (1532, 0.5), (1664, 0.5), (2044, 0.5), (4208, 0.5), (6130, 0.5),
    (11648, 0.5), (11776, 0.5),
    # ratio 1/4: up to 1408 rows refused, 1520 the shortest; 10240 the longest without moments in the workspace, and the next
    (1396, 0.25), (1400, 0.25), (1408, 0.25), (1520, 0.25), (1524, 0.25), (2048, 0.25), (2172, 0.25), (4092, 0.25), (6140, 0.25),
    (10240, 0.25), (10352, 0.25), (13184, 0.25),
]
REFUSED = [(1000, 0.5), (11776, 0.5), (1396, 0.25), (1400, 0.25), (1408, 0.25), (10352, 0.25), (13184, 0.25)]


def _by_units(wl):
    L = binding.Layout()
    L.dtype, L.n_layers, L.batch, L.token_capacity, L.stride_token = fk.BF16, 1, 1, wl.window, wl.head_dim
    return fk.compress_kernel(L, 1, wl.head_dim, wl.window, wl.n_sink, wl.retain_ratio) == "k_nearfar_units"


def _workload(span, ratio, **kw):
    args = dict(n_layers=1, batch=1, n_heads=1, head_dim=32, window=span + 4, retain_ratio=ratio, total_tokens=span + 4)
    args.update(kw)
    return synth.small(synth.WORKLOADS["llama2_7b_layer"], **args)


@pytest.mark.parametrize("span,ratio", SPANS)
def test_units_every_element(span, ratio):
    wl = _workload(span, ratio)
    _say(f"units {span} {ratio}")
    assert _by_units(wl) == ((span, ratio) not in REFUSED)
    k, v = _mk(wl, seed=span, capacity=span + 20, cur_len=span + 9)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, span + 9)
    assert rc == 0
    worst = _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, span + 9, TOL_BF16)
    assert worst <= 5e-3                                    # exact entries in 16 bits, as in test_gpu_nearfar


@pytest.mark.parametrize("span,ratio,heads", [(1020, 0.5, 300), (4092, 0.5, 140), (4092, 0.25, 140)])
def test_units_many_tasks(span, ratio, heads):
    """Ring, held blocks and moments handed from task to task, in both directions round the ring."""
    wl = _workload(span, ratio, n_heads=heads, head_dim=64)
    assert _by_units(wl)
    k, v = _mk(wl, seed=7)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, wl.window)
    assert rc == 0
    sub = synth.small(wl, n_heads=3)
    for h in (0, heads // 2, heads - 3):
        pick = (slice(None), slice(None), slice(h, h + 3))
        _check_all_heads(sub, k0[pick], v0[pick], k.cpu()[pick], v.cpu()[pick], tap.cpu()[(slice(None),) + pick], p, wl.window, TOL_BF16)
    # every head alone: the same bits
    for h in (1, heads // 3, heads - 1):
        kh, vh = k0[:, :, h:h + 1].cuda(), v0[:, :, h:h + 1].cuda()
        _run(kh, vh, synth.small(wl, n_heads=1), wl.window, tap=False)
        assert torch.equal(kh[:, :, :, :p.new_len], k[:, :, h:h + 1, :p.new_len])
        assert torch.equal(vh[:, :, :, :p.new_len], v[:, :, h:h + 1, :p.new_len])


def test_units_token_major():
    wl = _workload(2044, 0.5, n_heads=3, head_dim=64)
    assert _by_units(wl)
    k, v = _mk(wl, seed=3)
    kt, vt = (x.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4) for x in (k, v))
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    rc_t, _, _ = _run(kt, vt, wl, wl.window, tap=False)
    assert rc == rc_t == 0
    assert torch.equal(k[:, :, :, :p.new_len], kt[:, :, :, :p.new_len]) and torch.equal(v[:, :, :, :p.new_len], vt[:, :, :, :p.new_len])


@pytest.mark.parametrize("row", [0, 3, 63, 64, 1000, 4035, 4091])
def test_units_nan_stays_in_its_channel(row):
    """... also where it comes from a row whose image the first or the last leaf holds."""
    wl = _workload(4092, 0.5, head_dim=64)
    assert _by_units(wl)
    k, v = _mk(wl, seed=4)
    clean = k.clone()
    k[0, 0, 0, 4 + row, 17] = float("nan")
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    _run(clean, v.clone(), wl, wl.window, tap=False)
    assert rc == 0
    got = k[0, 0, 0, 4:p.new_len].float()
    ok = [c for c in range(64) if c != 17]
    assert not torch.isfinite(got[:, 17]).any()
    assert torch.equal(got[:, ok], clean[0, 0, 0, 4:p.new_len].float()[:, ok])


@pytest.mark.parametrize("rho", [0.0, 0.9])
@pytest.mark.parametrize("span,ratio", [(1020, 0.5), (1532, 0.25), (4092, 0.25), (8188, 0.5), (10236, 0.25), (11260, 0.25)])
def test_units_error_bound(span, ratio, rho):
    """rms distance from 64 bits before the result is rounded, over the rms of the result.  What a tile at a time reached at these spans
    and 200 others: 1.34e-4 to 1.55e-4 on white rows, 5.0e-5 to 8.2e-5 on autoregressive ones; a bound of 1.6e-4 and 9e-5."""
    x = np.random.default_rng(span).standard_normal((2, span, 32))
    for t in range(1, span):
        x[:, t] += rho * x[:, t - 1]
    rows = torch.from_numpy(x).to(torch.bfloat16)
    wl = _workload(span, ratio, n_sink=0, window=span, total_tokens=span)
    assert _by_units(wl) == ((span, ratio) != (11260, 0.25))        # that one in two parts, see test_gpu_nearfar_spill
    k, v = (rows[i].to("cuda").reshape(1, 1, 1, span, 32).clone() for i in range(2))
    rc, p, tap = _run(k, v, wl, span)
    assert rc == 0
    ref = np.stack([orc.compress_span(f64(rows[i]), p.retained_len) for i in range(2)])
    err = np.sqrt(((f64(tap).reshape(ref.shape) - ref) ** 2).mean() / (ref ** 2).mean())
    _say(f"units span {span} ratio {ratio} rho {rho}: rms error {err:.3e}")
    assert err <= (9e-5 if rho else 1.6e-4)
