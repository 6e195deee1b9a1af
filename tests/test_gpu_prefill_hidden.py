"""Chunk-wise attention of few queries over cached rows that are not finite: what a query does not see (later tokens of the chunk, rows past the end
of the cache) leaves its results as they are, and what it sees takes it to infinity or NaN in the channels that hold such a value and in no other."""
import numpy as np
import pytest
import torch

from _util import bf16_ulp, f64
from test_gpu_attend import TOL_ATT_F32
from test_gpu_prefill import _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu
CHANNEL = 17


def _same(got, want, vmax):
    """Both are a rounding to bf16 of sums in fp32 of the same terms, each within TOL_ATT_F32 of the largest value for scores of up to 8 units."""
    return (np.abs(got - want) <= bf16_ulp(want) * 1.001 + 2 * TOL_ATT_F32 * 4 * vmax).all()


@pytest.mark.parametrize("hkv,group,q_len,cur_len", [
    (1, 1, 1, 300),          # one query, the last step of 12 rows
    (2, 4, 1, 65),           # four heads, one row in the last step
    (2, 2, 5, 300),          # a set of four over the end of a head's chunk of queries
    (1, 3, 21, 2113),        # sets of the middle, in several chunks of rows
    (1, 1, 33, 100),         # more queries than rows in a step
    (1, 1, 64, 64),          # all of the cache
    (1, 1, 64, 2113),
    (1, 8, 5, 333),
    (3, 5, 3, 97),           # fewer queries than a set has
])
def test_values_of_rows_that_a_query_does_not_see(hkv, group, q_len, cur_len):
    wl = _wl(hkv=hkv, hq=hkv * group, cap=cur_len + 3)
    q, k, v = _mk(wl, cur_len, q_len, seed=cur_len + q_len)
    q *= 0.25                                          # weights well above zero for all rows
    vmax = float(v[..., :cur_len, :].float().abs().max())
    clean = f64(_run(q, k, v, wl, cur_len)[0].cpu())
    assert np.isfinite(clean).all()
    keep = [c for c in range(wl.head_dim) if c != CHANNEL]
    for back in sorted({0, 1, 2, 3, q_len // 2, q_len - 1} & set(range(q_len))):
        row = cur_len - 1 - back
        for value in (float("inf"), float("-inf"), float("nan")):
            _say(f"hidden values {hkv} x {group} x {q_len} over {cur_len}: row {row}, {value}")
            v2 = v.clone()
            v2[..., row, CHANNEL] = value
            out = f64(_run(q, k, v2, wl, cur_len)[0].cpu())
            before, after = slice(0, q_len - 1 - back), slice(q_len - 1 - back, q_len)     # queries that do not see it, and that do
            assert _same(out[..., keep], clean[..., keep], vmax)
            assert _same(out[..., before, CHANNEL], clean[..., before, CHANNEL], vmax)
            seen = out[..., after, CHANNEL]
            assert np.isnan(seen).all() if np.isnan(value) else (seen == value).all()


@pytest.mark.parametrize("hkv,group,q_len,cur_len", [(2, 2, 5, 300), (1, 1, 64, 2113), (1, 3, 21, 97)])
def test_keys_of_rows_that_a_query_does_not_see(hkv, group, q_len, cur_len):
    wl = _wl(hkv=hkv, hq=hkv * group, cap=cur_len)
    q, k, v = _mk(wl, cur_len, q_len, seed=cur_len)
    vmax = float(v.float().abs().max())
    clean = f64(_run(q, k, v, wl, cur_len)[0].cpu())
    for back in sorted({0, 1, q_len // 2}):
        k2 = k.clone()
        k2[..., cur_len - 1 - back, :] = float("nan")
        out = f64(_run(q, k2, v, wl, cur_len)[0].cpu())
        assert _same(out[..., :q_len - 1 - back, :], clean[..., :q_len - 1 - back, :], vmax)
        assert np.isnan(out[..., q_len - 1 - back:, :]).all()
