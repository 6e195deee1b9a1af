"""GPU parity of decode attention with four query heads handled together (softmax by quads of lanes, weighted sums on the matrix cores) against
the fp64 oracle: head sizes with 8, 16 and 32 lanes to a row, both cache types, one and two groups of four heads, heads of very
different scores whose reference points move at different rows, values that are not finite."""
import math

import numpy as np
import pytest
import torch

from oracle import attend_oracle as att

from _util import bf16_ulp, f64
from test_gpu_attend import TOL_ATT_F32, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


def _check_heads(q, k, v, out, lse, wl, b, cur_len):
    """One sequence, every head by itself.  A score s is a sum of d fp32 products, off by up to some 2^-22 |s|, and so is the weight, relatively: the
    tolerance of these tests, 2e-6 of the largest value, stands for scores of up to 8 units, and a head whose scores go beyond that has as much
    more as the largest of them in 64 bits says."""
    d, group = wl.head_dim, wl.q_heads // wl.n_heads
    for h in range(wl.q_heads):
        kk, vv = f64(k[0, b, h // group, :cur_len]), f64(v[0, b, h // group, :cur_len])
        qq = f64(q[0, b, h])
        ref, rlse = att.attend_decode_head(qq, kk, vv, cur_len, None, wl.rope_base)
        scores = att.rope_rotate(kk, np.arange(cur_len), wl.rope_base) @ att.rope_rotate(qq, cur_len - 1, wl.rope_base) / math.sqrt(d)
        tol = TOL_ATT_F32 * max(1.0, float(np.abs(scores).max()) / 8.0) * float(np.abs(vv).max())
        bound = tol + (0.5 * bf16_ulp(ref) * 1.001 if wl.dtype == torch.bfloat16 else 0.0)
        err = np.abs(f64(out[0, b, h]) - ref)
        assert (err <= bound).all(), (b, h, float(np.abs(scores).max()), float((err / bound).max()))
        assert abs(float(lse[0, b, h]) - rlse) <= 2e-5 * (1.0 + abs(rlse)), (b, h)


def _ramp(q, k, cur_len):
    """Scores that rise along the rows, in some heads by far more than in others."""
    k[:, :, :, :cur_len] *= torch.linspace(0.2, 2.0, cur_len, device=k.device).view(1, 1, 1, -1, 1).to(k.dtype)
    q *= torch.tensor([0.01, 2.0, 0.3, 1.0, 0.0, 1.5, 0.7, 2.5], device=q.device).repeat(q.shape[2] // 8).view(1, 1, -1, 1).to(q.dtype)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("cur_len,batch", [(1, 1), (31, 3), (33, 1), (700, 2), (2051, 1), (300, 200)])
@pytest.mark.parametrize("hq", [8, 16])
def test_quads(hq, cur_len, batch, d, dtype):
    wl = _wl(d=d, hkv=2, hq=hq, batch=batch, cap=cur_len + 3, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    _ramp(q, k, cur_len)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"quads {hq} {cur_len} {batch} {d} {dtype}: n_split {p.n_split}")
    assert p.heads_together == 4
    q, k, v, out, lse = (t.cpu() for t in (q, k, v, out, lse))
    for b in sorted({0, batch // 2, batch - 1}):
        _check_heads(q, k, v, out, lse, wl, b, cur_len)


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


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d,cur_len", [(64, 4097), (64, 4225), (128, 2047), (128, 2049), (128, 2113), (256, 1025), (256, 2081)])
def test_quads_long_chunks(d, cur_len, dtype):
    """Whole sequences in one chunk each, below and beyond the 64 steps between exact angles: an odd and an even number of steps, a last step of one row."""
    batch = 256
    wl = _wl(d=d, hkv=2, hq=8, batch=batch, cap=cur_len, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    _ramp(q, k, cur_len)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"quads, long chunks {cur_len} {d} {dtype}: n_split {p.n_split}")
    assert p.n_split == 1
    q, k, v, out, lse = (t[:, [0, 255]].cpu() for t in (q, k, v, out, lse))
    for b in range(2):
        _check_heads(q, k, v, out, lse, wl, b, cur_len)
