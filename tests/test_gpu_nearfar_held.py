"""GPU tests of the units of leaves that the movers of the form by units hold: 1 to 6 of them, at every place that a unit's first leaf can have
in its block, next to each other and apart, over several tasks of a workgroup."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding

from _util import TOL_BF16
from test_gpu_nearfar_units import _workload
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

# (span, ratio): ring slots, held units, first leaf of the first, leaves from each to the next
SPANS = {(2300, 0.5): (14, 1, 14, 4),
         (2944, 0.5): (14, 2, 14, 4),
         (3452, 0.5): (14, 3, 14, 4),
         (4092, 0.5): (13, 4, 13, 4),
         (5632, 0.5): (12, 4, 16, 8),
         (7160, 0.5): (11, 4, 15, 8),
         (9472, 0.5): (10, 4, 22, 16),
         (10364, 0.5): (9, 4, 21, 16),
         (2432, 0.25): (15, 1, 15, 4),
         (3196, 0.25): (14, 2, 14, 4),
         (4348, 0.25): (14, 5, 14, 4),
         (4736, 0.25): (13, 6, 13, 4),
         (6140, 0.25): (12, 6, 12, 4),
         (7296, 0.25): (11, 6, 11, 4),
         (8700, 0.25): (10, 6, 14, 8)}
assert {first % 4 for _, _, first, _ in SPANS.values()} == {0, 1, 2, 3} and {held for _, held, _, _ in SPANS.values()} == {1, 2, 3, 4, 5, 6}


@pytest.mark.parametrize("span,ratio", SPANS)
def test_held_units(span, ratio):
    """Head-tensors are one and the same but for a power of two, which goes through every sum and rounding: so what a task finds of the one
    before it shows."""
    heads = 600
    _say(f"held units {span} {ratio}")
    one = _workload(span, ratio)
    L = binding.Layout()
    L.dtype, L.n_layers, L.batch, L.token_capacity, L.stride_token = fk.BF16, 1, 1, one.window, one.head_dim
    assert fk.compress_ring(L, 1, one.head_dim, one.window, one.n_sink, one.retain_ratio) == SPANS[span, ratio]
    k1, v1 = _mk(one, seed=span)
    scale = (2.0 ** (torch.arange(heads) % 7)).view(1, 1, heads, 1, 1).to("cuda", torch.bfloat16)
    k, v = k1 * scale, v1 * scale
    before = k1.cpu().clone(), v1.cpu().clone()
    rc, p, tap = _run(k1, v1, one, one.window)
    assert rc == 0
    _check_all_heads(one, *before, k1.cpu(), v1.cpu(), tap.cpu(), p, one.window, TOL_BF16)
    rc, _, _ = _run(k, v, _workload(span, ratio, n_heads=heads), one.window, tap=False)
    assert rc == 0
    for got, want in ((k, k1), (v, v1)):
        assert torch.equal(got[:, :, :, :p.new_len], want[:, :, :, :p.new_len] * scale)
