"""GPU parity of the near/far form against the fp64 CPU oracle, every element: spans around the edges of its leaves
(128 rows), blocks (512) and ring, ratios on both sides of its window sizes, odd lengths, shared and separate tables."""
import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from oracle import freqkv_oracle as orc

from _util import TOL_BF16, f64
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

CASES = [
    # (layers, batch, heads, d, span, ratio)
    (1, 1, 1, 32, 128, 0.5), (1, 1, 1, 32, 129, 0.5), (1, 1, 1, 64, 191, 0.97), (1, 1, 1, 32, 256, 0.5),
    (1, 1, 2, 32, 257, 0.25), (1, 1, 1, 32, 383, 0.2), (1, 1, 1, 32, 384, 0.25), (1, 1, 1, 32, 511, 0.44),
    (1, 1, 1, 32, 512, 0.45), (1, 1, 1, 32, 513, 0.6), (2, 1, 9, 32, 640, 0.5), (1, 1, 1, 32, 1000, 0.999),
    (1, 1, 1, 96, 1024, 0.5), (1, 1, 1, 32, 1025, 0.5), (1, 1, 1, 32, 2048, 0.25), (1, 1, 1, 32, 2100, 0.375),
    (1, 1, 1, 32, 4096, 0.5), (1, 1, 1, 32, 4864, 0.5), (1, 1, 1, 32, 4993, 0.5), (1, 1, 1, 32, 6083, 0.5), (1, 1, 1, 32, 8192, 0.2), (1, 1, 1, 32, 8192, 0.9),
    (1, 1, 1, 32, 12284, 0.5), (1, 3, 100, 32, 1536, 0.5), (1, 3, 60, 32, 5377, 0.6),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_nearfar_every_element(case):
    layers, batch, heads, d, span, ratio = case
    wl = synth.small(synth.WORKLOADS["llama2_7b_layer"], n_layers=layers, batch=batch, n_heads=heads, head_dim=d,
                     window=span + 3, n_sink=3, retain_ratio=ratio, total_tokens=span + 3)
    _say(f"near/far {case}")
    k, v = _mk(wl, seed=span + d, capacity=span + 9)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, wl.window)
    assert rc == 0
    if heads > 50:                                          # more tasks than workgroups: a few head-tensors of the many
        sub = synth.small(wl, batch=1, n_heads=4)
        pick = (slice(None), slice(2, 3), slice(heads - 4, heads))
        _check_all_heads(sub, k0[pick], v0[pick], k.cpu()[pick], v.cpu()[pick], tap.cpu()[(slice(None),) + pick], p, wl.window, TOL_BF16)
        return
    worst = _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, wl.window, TOL_BF16)
    assert worst <= 5e-3                                    # exact entries in 16 bits: closer than the general tolerance


def test_nearfar_nan_stays_in_its_channel():
    wl = synth.small(synth.WORKLOADS["llama2_7b_layer"], n_heads=1, head_dim=64, window=2052)
    k, v = _mk(wl, seed=4)
    clean = k.clone()
    k[0, 0, 0, 1000, 17] = float("nan")
    k[0, 0, 0, 2051, 40] = float("inf")
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    _run(clean, v.clone(), wl, wl.window, tap=False)
    assert rc == 0
    got = k[0, 0, 0, 4:p.new_len].float()
    ok = [c for c in range(64) if c not in (17, 40)]
    assert not torch.isfinite(got[:, 17]).any() and not torch.isfinite(got[:, 40]).any()
    assert torch.equal(got[:, ok], clean[0, 0, 0, 4:p.new_len].float()[:, ok])


@pytest.mark.parametrize("rho", [0.0, 0.9])
@pytest.mark.parametrize("span,ratio", [(1020, 0.25), (2044, 0.25), (8188, 0.25), (6083, 0.25), (4095, 0.2), (2996, 0.3125), (6083, 0.45),
                                        (4999, 0.5), (4092, 0.5), (3000, 0.9)])
def test_nearfar_is_no_further_off_than_the_matrix_forms(span, ratio, rho):
    """Before the result is rounded to bf16: rms distance from 64 bits, white rows and rows that are correlated along the
    tokens.  The matrix forms round every entry once to fp16."""
    wl = synth.small(synth.WORKLOADS["llama2_7b_layer"], n_heads=1, head_dim=64, window=span, n_sink=0, retain_ratio=ratio,
                     total_tokens=span)
    x = np.random.default_rng(span).standard_normal((2, span, 64))
    for t in range(1, span):
        x[:, t] += rho * x[:, t - 1]
    rows = torch.from_numpy(x).to(torch.bfloat16)
    err = []
    for flags in (0, fk.FLAG_DENSE):
        k, v = (rows[i].to("cuda").reshape(1, 1, 1, span, 64).clone() for i in range(2))
        rc, p, tap = _run(k, v, wl, span, flags=flags)
        assert rc == 0
        ref = np.stack([orc.compress_span(f64(rows[i]), p.retained_len) for i in range(2)])
        err.append(np.sqrt(((f64(tap).reshape(ref.shape) - ref) ** 2).mean() / (ref ** 2).mean()))
    _say(f"near/far span {span} ratio {ratio} rho {rho}: rms error {err[0]:.3e}, matrix form {err[1]:.3e}")
    assert err[0] <= err[1]


@pytest.mark.parametrize("layers,lens", [(1, [140, 133, 400, 132, 12]), (33, [132, 133, 250, 3, 132])])
def test_nearfar_ragged_is_each_sequence_alone(layers, lens):
    """One pass over all due sequences: tails longer than the rows set free, more slabs than one pass holds."""
    wl = synth.small(synth.WORKLOADS["llama2_7b_layer"], n_layers=layers, batch=5, n_heads=3, head_dim=32, window=132)
    k, v = _mk(wl, seed=5, capacity=max(lens) + 3, cur_len=max(lens) + 3)
    k0, v0 = k.clone(), v.clone()
    L = binding.layout_for(k)
    _, p = fk.plan(L, 3, 32, 132, 132, wl.n_sink, 0.5)
    ws = torch.empty(max(p.workspace_bytes, 256), dtype=torch.uint8, device=k.device)
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    _, new = fk.compress_ragged(k, v, L, 3, 32, lens, 132, wl.n_sink, 0.5)
    for b, n in enumerate(lens):
        kb, vb = k0[:, b:b + 1].clone(), v0[:, b:b + 1].clone()
        if n >= 132:
            _run(kb, vb, synth.small(wl, batch=1), n, tap=False)
        assert new[b] == (n if n < 132 else n - 132 + wl.n_sink + p.retained_len)
        for got, want, before in ((k, kb, k0), (v, vb, v0)):
            assert torch.equal(got[:, b, :, :new[b]], want[:, 0, :, :new[b]])
            assert torch.equal(got[:, b, :, n:], before[:, b, :, n:])
