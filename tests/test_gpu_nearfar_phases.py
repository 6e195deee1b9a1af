"""GPU tests of the moments' tables that all leaves but the last share (windows of 2 leaves, exact entries of their own per tile): last leaves
of 1 to 128 rows, spans of 1 leaf and a row up to those that use the workspace; many tasks to a workgroup."""
import numpy as np
import pytest
import torch

from paper_2505_00570_amd import synth

from oracle import freqkv_oracle as orc

from _util import TOL_BF16, f64
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _workload(span, ratio, **kw):
    args = dict(n_layers=1, batch=1, n_heads=1, head_dim=32, n_sink=0, window=span, retain_ratio=ratio, total_tokens=span)
    args.update(kw)
    return synth.small(synth.WORKLOADS["llama2_7b_layer"], **args)


# rms distance from 64 bits before the result is rounded, over the rms of the result, with a table of its own for each leaf
WITH_OWN_TABLES = [(257, 0.5, 0.870e-4), (511, 0.6, 1.028e-4), (769, 0.5, 1.254e-4), (1151, 0.75, 1.071e-4), (2049, 0.9, 1.012e-4),
                   (4999, 0.5, 1.466e-4), (8191, 0.75, 1.194e-4), (13999, 0.5, 1.508e-4), (14813, 0.6, 0.832e-4)]


@pytest.mark.parametrize("span,ratio,own", WITH_OWN_TABLES)
def test_error_is_that_of_a_table_per_leaf(span, ratio, own):
    """Sums are rounded at other places.  The rms of N independent errors drawn anew moves by 1 / sqrt(2 N) of itself: twice that over it at most, and 0.1 % for
    the digits of the figures above."""
    rows = torch.from_numpy(np.random.default_rng(span).standard_normal((2, span, 64))).to(torch.bfloat16)
    k, v = (rows[i].to("cuda").reshape(1, 1, 1, span, 64).clone() for i in range(2))
    rc, p, tap = _run(k, v, _workload(span, ratio, head_dim=64), span)
    assert rc == 0
    ref = np.stack([orc.compress_span(f64(rows[i]), p.retained_len) for i in range(2)])
    err = np.sqrt(((f64(tap).reshape(ref.shape) - ref) ** 2).mean() / (ref ** 2).mean())
    _say(f"phases {span} {ratio}: rms error {err:.3e} of {own:.3e}")
    assert err <= (1.001 + 2.0 / np.sqrt(2.0 * ref.size)) * own


@pytest.mark.parametrize("span,ratio", [(129, 0.6), (255, 0.9), (256, 0.6), (1281, 0.6), (1407, 0.6), (1600, 0.7), (3073, 0.45), (3199, 0.95)])
def test_last_leaf(span, ratio):
    """Every element; head-tensors that are the same but for a power of two, several to a workgroup, come out the same but for it."""
    heads = 600
    one = _workload(span, ratio)
    k1, v1 = _mk(one, seed=span)
    scale = (2.0 ** (torch.arange(heads) % 7)).view(1, 1, heads, 1, 1).to("cuda", torch.bfloat16)
    k, v = k1 * scale, v1 * scale
    before = k1.cpu().clone(), v1.cpu().clone()
    rc, p, tap = _run(k1, v1, one, span)
    assert rc == 0
    _check_all_heads(one, *before, k1.cpu(), v1.cpu(), tap.cpu(), p, span, TOL_BF16)
    rc, _, _ = _run(k, v, _workload(span, ratio, n_heads=heads), span, tap=False)
    assert rc == 0
    for got, want in ((k, k1), (v, v1)):
        assert torch.equal(got[:, :, :, :p.new_len], want[:, :, :, :p.new_len] * scale)
