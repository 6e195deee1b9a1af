"""GPU parity of the near/far form on spans of up to 3 blocks (1536 rows), none of which is far from any group, and on the first longer
ones, against the fp64 CPU oracle, every element: 1 to 3 blocks, windows of 2 and 3 leaves, each count of second parts, tables that repeat
and that do not; one step of tiles and many; tasks handed on with the ring turning either way."""
import pytest
import torch

from paper_2505_00570_amd import synth

from _util import TOL_BF16
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _workload(span, ratio, **kw):
    args = dict(n_layers=1, batch=1, n_heads=1, head_dim=32, window=span + 4, retain_ratio=ratio, total_tokens=span + 4)
    args.update(kw)
    return synth.small(synth.WORKLOADS["llama2_7b_layer"], **args)


@pytest.mark.parametrize("span", [128, 129, 511, 512, 513, 1024, 1025, 1535, 1536, 1537])
@pytest.mark.parametrize("ratio", [0.25, 0.36, 0.5, 0.7])
def test_short_every_element(span, ratio):
    wl = _workload(span, ratio)
    _say(f"short {span} {ratio}")
    k, v = _mk(wl, seed=span, capacity=span + 20, cur_len=span + 9)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, span + 9)
    assert rc == 0 and p.runs == 7
    assert _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, span + 9, TOL_BF16) <= 5e-3


@pytest.mark.parametrize("span,ratio", [(131, 0.5), (300, 0.25), (700, 0.6), (1530, 0.36)])
def test_short_many_tasks(span, ratio):
    """Several tasks to a workgroup: every head alone gives the same bits."""
    wl = _workload(span, ratio, n_heads=500)
    k, v = _mk(wl, seed=9)
    k0, v0 = k.clone(), v.clone()
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    assert rc == 0
    for h in (0, 77, 300, 499):
        kh, vh = k0[:, :, h:h + 1].clone(), v0[:, :, h:h + 1].clone()
        _run(kh, vh, synth.small(wl, n_heads=1), wl.window, tap=False)
        assert torch.equal(kh[:, :, :, :p.new_len], k[:, :, h:h + 1, :p.new_len])
        assert torch.equal(vh[:, :, :, :p.new_len], v[:, :, h:h + 1, :p.new_len])
