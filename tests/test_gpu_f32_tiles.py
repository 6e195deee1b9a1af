"""GPU parity of the fp32 contraction in tiles of 16 and of 32, against the fp64 CPU oracle, every element: contraction lengths of every
remainder to 4 and shorter than 4, shares of a wave that end within a unit of loads, both sides of the rule between the tiles, more slabs
than fit the short table of pointers; and the same bits from both."""
import pytest
import torch

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


@pytest.mark.parametrize("span,ratio", [(508, 0.5), (510, 0.5), (512, 0.5), (514, 0.5), (2044, 0.5), (1500, 0.3),      # folded, every remainder to 4
                                        (509, 0.5), (511, 0.7), (510, 0.9), (512, 0.3), (1023, 0.5)])                  # plain
def test_bits_do_not_depend_on_the_columns_of_a_pass(span, ratio):
    """All heads in one call, one at a time, and a slab to a pass in the smallest workspace: different tiles, the same bits."""
    heads = 20
    wl = synth.small(synth.WORKLOADS["tiny"], n_layers=1, batch=1, n_heads=heads, head_dim=64, window=span + 1, n_sink=1, retain_ratio=ratio,
                     total_tokens=span + 1)
    one = synth.small(wl, n_heads=1)
    k, v = _mk(wl, seed=span)
    ka, va, kb, vb = (t.clone() for t in (k, v, k, v))
    rc, p, _ = _run(ka, va, wl, span + 1, tap=False)
    assert rc == 0 and p.variant == 3
    rows = -(-p.retained_len // (64 if p.retained_len % 2 == 0 and span % 2 == 0 else 32))
    assert rows * (2 * heads * 64 // 32) > 192 >= rows * (2 * 64 // 32)              # tiles of 32 and of 16
    assert _run(kb, vb, wl, span + 1, tap=False, ws_bytes=p.workspace_min_bytes)[0] == 0
    for h in range(heads):
        kh, vh = k[:, :, h:h + 1].clone(), v[:, :, h:h + 1].clone()
        assert _run(kh, vh, one, span + 1, tap=False)[0] == 0
        assert torch.equal(ka[:, :, h], kh[:, :, 0]) and torch.equal(va[:, :, h], vh[:, :, 0]), h
    assert torch.equal(ka, kb) and torch.equal(va, vb)
