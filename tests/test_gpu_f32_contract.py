"""GPU parity of the fp32 contraction against the fp64 CPU oracle, every element: folded and plain spans, remainders of its
tiles (32 rows, 32 columns) and of its contraction slices, four waves to a tile, a whole pass of both kinds."""
import pytest

from paper_2505_00570_amd import synth

from _util import TOL_F32
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

CASES = [
    # (layers, heads, d, window, n_sink, ratio)
    (1, 1, 8, 9, 1, 0.5), (1, 1, 8, 14, 4, 0.3), (1, 1, 8, 67, 4, 0.5), (1, 1, 64, 68, 4, 0.5), (1, 1, 40, 70, 4, 0.97),
    (1, 1, 64, 133, 4, 0.25), (2, 3, 24, 200, 0, 0.5), (1, 1, 64, 512, 4, 0.5), (1, 2, 128, 515, 4, 0.5), (1, 1, 64, 2048, 4, 0.1),
    (2, 8, 128, 1028, 4, 0.5), (1, 8, 128, 619, 4, 0.5), (4, 8, 72, 1030, 4, 0.52),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_f32_contraction_every_element(case):
    layers, heads, d, window, sinks, ratio = case
    wl = synth.small(synth.WORKLOADS["tiny"], n_layers=layers, batch=1, n_heads=heads, head_dim=d, window=window,
                     n_sink=sinks, retain_ratio=ratio, total_tokens=window + 5)
    _say(f"fp32 {case}")
    k, v = _mk(wl, seed=window + d, capacity=window + 9, cur_len=window + 5)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, wl.window + 5)
    assert rc == 0
    _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, wl.window + 5, TOL_F32)
