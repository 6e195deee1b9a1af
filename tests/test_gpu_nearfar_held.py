"""GPU tests of the units of leaves that the movers of the form by units hold: 1 to 6 of them, at every place that a unit's first leaf can have
in its block, next to each other and apart, over several tasks of a workgroup."""
import pytest
import torch

from _util import TOL_BF16
from test_gpu_nearfar_units import _by_units, _workload
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu

# (span, ratio): ring slots, held units
SPANS = [(2300, 0.5),      # 14, 1
         (2944, 0.5),      # 14, 2
         (3452, 0.5),      # 14, 3
         (4092, 0.5),      # 13, 4
         (5632, 0.5),      # 12, 4, every second one from the second on
         (7160, 0.5),      # 11, 4
         (9472, 0.5),      # 10, 4, every fourth
         (10364, 0.5),     # 9, 4
         (2432, 0.25),     # 15, 1
         (3196, 0.25),     # 14, 2
         (4348, 0.25),     # 14, 5
         (4736, 0.25),     # 13, 6
         (6140, 0.25),     # 12, 6
         (7296, 0.25),     # 11, 6
         (8700, 0.25)]     # 10, 6, every second


@pytest.mark.parametrize("span,ratio", SPANS)
def test_held_units(span, ratio):
    """Head-tensors are one and the same but for a power of two, which goes through every sum and rounding: so what a task finds of the one
    before it shows."""
    heads = 600
    _say(f"held units {span} {ratio}")
    one = _workload(span, ratio)
    assert _by_units(one)
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
