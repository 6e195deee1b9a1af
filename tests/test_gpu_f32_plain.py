"""GPU parity of the unfolded fp32 contraction against the fp64 CPU oracle, every element: slices of one wave (a quarter of the span, two
rows a step) around one and two sets of 16 steps, and with last sets of one step and of none."""
import pytest

from paper_2505_00570_amd import synth

from _util import TOL_F32
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span", [3, 121, 127, 129, 130, 136, 249, 255, 257, 258, 265, 383, 385, 513, 1025])
def test_plain_slices(span):
    wl = synth.small(synth.WORKLOADS["tiny"], n_layers=1, batch=1, n_heads=1, head_dim=40, window=span, n_sink=0,
                     retain_ratio=(span // 2 | 1) / span + 1e-9, total_tokens=span)
    _say(f"fp32 plain {span}")
    k, v = _mk(wl, seed=span)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, span)
    assert rc == 0 and p.retained_len % 2 == 1
    _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, span, TOL_F32)
