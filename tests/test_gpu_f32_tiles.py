"""GPU parity of the fp32 contraction in tiles of 16 and of 32, against the fp64 CPU oracle, every element: contraction lengths of every
remainder to 4 and shorter than 4, shares of a wave that end within a unit of loads, both sides of the rule between the tiles, more slabs
than fit the short table of pointers."""
import pytest

from paper_2505_00570_amd import synth

from _util import TOL_F32
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

CASES = [
    # (layers, heads, d, span, ratio)
    # folded: contraction lengths 1 to 9, 62 to 66, 126 to 129
    *[(1, 1, 8, 2 * k, 0.5 if k % 2 == 0 else (k - 1) / (2 * k) + 1e-9) for k in (2, 3, 4, 5, 6, 7, 8, 9)],
    *[(1, 1, 24, 2 * k, 0.5 if k % 2 == 0 else (k - 1) / (2 * k) + 1e-9) for k in (62, 63, 64, 65, 66, 126, 127, 128, 129)],
    # plain, the same lengths
    *[(1, 1, 16, n, (n // 2 | 1) / n + 1e-9) for n in (3, 5, 6, 7, 9, 62, 63, 64, 65, 66)],
    # 192 workgroups of 32 x 32 and 193 or more: 6 x 32 tiles and 7 x 32, 12 x 16 and 13 x 16 (plain)
    (1, 4, 128, 768, 0.5), (1, 4, 128, 776, 0.5), (1, 2, 128, 767, 0.5), (1, 2, 128, 771, 0.5),
    # 8 slabs and 10, in both tiles
    (4, 1, 8, 100, 0.5), (5, 1, 8, 100, 0.5), (5, 1, 8, 101, 0.5), (5, 4, 128, 300, 0.5), (5, 4, 128, 301, 0.5),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_f32_tiles_every_element(case):
    layers, heads, d, span, ratio = case
    wl = synth.small(synth.WORKLOADS["tiny"], n_layers=layers, batch=1, n_heads=heads, head_dim=d, window=span + 1,
                     n_sink=1, retain_ratio=ratio, total_tokens=span + 4)
    _say(f"fp32 tiles {case}")
    k, v = _mk(wl, seed=span + d, capacity=span + 9, cur_len=span + 4)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, span + 4)
    assert rc == 0
    _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, span + 4, TOL_F32)
