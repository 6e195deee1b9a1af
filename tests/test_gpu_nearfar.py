"""GPU parity of the near/far form against the fp64 CPU oracle, every element: spans around the edges of its leaves
(128 rows), blocks (512) and ring, ratios on both sides of its window sizes, odd lengths, shared and separate tables."""
import pytest
import torch

from paper_2505_00570_amd import synth

from _util import TOL_BF16
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

CASES = [
    # (layers, batch, heads, d, span, ratio)
    (1, 1, 1, 32, 128, 0.5), (1, 1, 1, 32, 129, 0.5), (1, 1, 1, 64, 191, 0.97), (1, 1, 1, 32, 256, 0.5),
    (1, 1, 2, 32, 257, 0.25), (1, 1, 1, 32, 383, 0.2), (1, 1, 1, 32, 384, 0.25), (1, 1, 1, 32, 511, 0.44),
    (1, 1, 1, 32, 512, 0.45), (1, 1, 1, 32, 513, 0.6), (2, 1, 9, 32, 640, 0.5), (1, 1, 1, 32, 1000, 0.999),
    (1, 1, 1, 96, 1024, 0.5), (1, 1, 1, 32, 1025, 0.5), (1, 1, 1, 32, 2048, 0.25), (1, 1, 1, 32, 2100, 0.375),
    (1, 1, 1, 32, 4096, 0.5), (1, 1, 1, 32, 6083, 0.5), (1, 1, 1, 32, 8192, 0.2), (1, 1, 1, 32, 8192, 0.9),
    (1, 1, 1, 32, 12284, 0.5), (1, 3, 100, 32, 1536, 0.5),
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
