"""GPU parity of decode attention with four query heads handled together (softmax by quads of lanes, weighted sums on the matrix cores) against
the fp64 oracle: head sizes with 8, 16 and 32 lanes to a row, both cache types, one and two groups of four heads, heads of very
different scores whose reference points move at different rows, values that are not finite."""
import pytest
import torch

import test_gpu_attend
from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


def _ramp(q, k, cur_len):
    """Scores that rise along the rows, in some heads by far more than in others."""
    k[:, :, :, :cur_len] *= torch.linspace(0.2, 2.0, cur_len, device=k.device).view(1, 1, 1, -1, 1).to(k.dtype)
    q *= torch.tensor([0.01, 2.0, 0.3, 1.0, 0.0, 1.5, 0.7, 2.5], device=q.device).repeat(q.shape[2] // 8).view(1, 1, -1, 1).to(q.dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("cur_len,batch", [(1, 1), (31, 3), (33, 1), (700, 2), (2051, 1), (300, 200)])
@pytest.mark.parametrize("hq", [8, 16])
def test_quads(hq, cur_len, batch, d, dtype, monkeypatch):
    wl = _wl(d=d, hkv=2, hq=hq, batch=batch, cap=cur_len + 3, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    _ramp(q, k, cur_len)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"quads {hq} {cur_len} {batch} {d} {dtype}: n_split {p.n_split}")
    assert p.heads_together == 4
    # A score s is a sum of d fp32 products, off by up to some 2^-22 |s|, and so is the weight, relatively; the tolerance of these tests stands
    # for scores of up to 8 units.  Here the rising ones reach more: the largest is at most the logarithm of their sum.
    monkeypatch.setattr(test_gpu_attend, "TOL_ATT_F32", test_gpu_attend.TOL_ATT_F32 * max(1.0, float(lse.abs().max()) / 8.0))
    for b in sorted({0, batch // 2, batch - 1}):
        s = slice(b, b + 1)
        _check(q[:, s], k[:, s], v[:, s], out[:, s], lse[:, s], _wl(d=d, hkv=2, hq=hq, cap=cur_len + 3, dtype=dtype), cur_len)


@pytest.mark.parametrize("d", [64, 128, 256])
def test_quads_keep_channels_and_heads_apart(d):
    """A value that is not finite stays in its channel, a query that is not finite in its head; the others keep their bits."""
    wl = _wl(d=d, hkv=2, hq=8, cap=500)
    q, k, v = _mk(wl, 500, seed=d)
    clean, _, _ = _run(q, k, v, wl, 500)
    v2, q2 = v.clone(), q.clone()
    v2[0, 0, 1, 123, 17] = float("inf")
    q2[0, 0, 2, 5] = float("nan")
    out, _, _ = _run(q, k, v2, wl, 500)
    keep = [c for c in range(d) if c != 17]
    assert not torch.isfinite(out[0, 0, 4:, 17].float()).any()
    assert torch.equal(out[0, 0, :4], clean[0, 0, :4]) and torch.equal(out[0, 0, 4:][:, keep], clean[0, 0, 4:][:, keep])
    out, _, _ = _run(q2, k, v, wl, 500)
    others = [h for h in range(8) if h != 2]
    assert torch.isnan(out[0, 0, 2].float()).all() and torch.equal(out[0, 0, others], clean[0, 0, others])
