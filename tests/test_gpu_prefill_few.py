"""Chunk-wise attention of few queries, which go as heads of a decode call: each query by itself against the fp64 oracle, at the edges of groups of
four, of chunks and of the causal end; and what the other way of such calls guarantees."""
import math

import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding
from oracle import attend_oracle as att

from _util import bf16_ulp, f64
from test_gpu_attend import TOL_ATT_F32
from test_gpu_prefill import _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


def _check_queries(q, k, v, out, lse, wl, layer, b, cur_len):
    """As in decode with four heads: 2e-6 of the largest value for scores of up to 8 units, and as much more as larger ones say; fp32 throughout,
    where operands of 11 bits would be some 1e-3 off."""
    d, q_len, group = wl.head_dim, q.shape[3], wl.q_heads // wl.n_heads
    for h in range(wl.q_heads):
        kk, vv = f64(k[layer, b, h // group, :cur_len]), f64(v[layer, b, h // group, :cur_len])
        turned = att.rope_rotate(kk, np.arange(cur_len), wl.rope_base)
        for i in range(q_len):
            pos = cur_len - q_len + i
            qq = f64(q[layer, b, h, i])
            ref, rlse = att.attend_decode_head(qq, kk, vv, pos + 1, pos, wl.rope_base, True)
            scores = turned[:pos + 1] @ att.rope_rotate(qq, pos, wl.rope_base) / math.sqrt(d)
            tol = TOL_ATT_F32 * max(1.0, float(np.abs(scores).max()) / 8.0) * float(np.abs(vv).max())
            err = np.abs(f64(out[layer, b, h, i]) - ref)
            assert (err <= tol + 0.5 * bf16_ulp(ref) * 1.001).all(), (h, i, float(err.max()))
            assert abs(float(lse[layer, b, h, i]) - rlse) <= 2e-5 * (1.0 + abs(rlse)), (h, i)


@pytest.mark.parametrize("cur_len", [5, 33, 300, 2113])
@pytest.mark.parametrize("hkv,group,q_len", [(2, 1, 1), (1, 1, 5), (2, 3, 5), (1, 4, 4), (3, 5, 3), (2, 8, 2), (1, 1, 17), (1, 8, 5), (1, 3, 21), (1, 1, 64)])
def test_few_queries(hkv, group, q_len, cur_len):
    """Groups of four that are full, and of one, two and three; more and fewer queries than the cache has rows ahead of them."""
    if q_len > cur_len:
        pytest.skip("more queries than rows")
    several = 2 if cur_len < 1000 else 1               # (of more groups over long caches fewer go this way)
    wl = _wl(hkv=hkv, hq=hkv * group, layers=several, batch=several, cap=cur_len + 5)
    q, k, v = _mk(wl, cur_len, q_len, seed=cur_len + q_len)
    out, lse, _ = _run(q, k, v, wl, cur_len)
    _say(f"few queries {hkv} x {group} x {q_len} over {cur_len}")
    q, k, v, out, lse = (t.cpu() for t in (q, k, v, out, lse))
    for layer, b in {(0, 0), (several - 1, several - 1)}:
        _check_queries(q, k, v, out, lse, wl, layer, b, cur_len)


@pytest.mark.parametrize("cur_len,q_len", [(2049, 3), (4161, 2)])
def test_few_queries_long_chunks(cur_len, q_len):
    """One chunk to a sequence, beyond the steps between exact angles."""
    wl = _wl(hkv=2, hq=2, batch=256, cap=cur_len)
    q, k, v = _mk(wl, cur_len, q_len, seed=cur_len)
    out, lse, _ = _run(q, k, v, wl, cur_len)
    _say(f"few queries, long chunks: {q_len} over {cur_len}")
    for b in (0, 255):
        cut = [t[:, b:b + 1].cpu() for t in (q, k, v, out, lse)]
        _check_queries(*cut, wl, 0, 0, cur_len)


def test_few_queries_without_rotary():
    wl = _wl(hkv=2, hq=4, cap=300)
    q, k, v = _mk(wl, 300, 6, seed=9)
    out, _, _ = _run(q, k, v, wl, 300, base=0.0)
    for h in range(4):
        ref, _ = att.attend_prefill(f64(q[0, 0].cpu()), f64(k[0, 0].cpu()), f64(v[0, 0].cpu()), 300, 1e4, rope=False)
        assert (np.abs(f64(out[0, 0].cpu()) - ref) <= 0.5 * bf16_ulp(ref) * 1.001 + TOL_ATT_F32 * float(v.float().abs().max())).all()


def test_few_queries_in_the_least_workspace():
    """The least workspace that the other way takes is enough; with a byte less the call is refused, as before."""
    wl = _wl(hkv=2, hq=8, cap=1000)
    q, k, v = _mk(wl, 1000, 4, seed=4)
    want, _, _ = _run(q, k, v, wl, 1000)
    least = 1000 * 64 * 8 + 2 * 2 * 32 * 32 * 128 * 2
    for size, ok in ((least, True), (least - 1, False)):
        L = binding.layout_for(k)
        ws = torch.empty(least, dtype=torch.uint8, device="cuda")
        L.workspace, L.workspace_bytes = ws.data_ptr(), size
        out = torch.full_like(q, float("nan"))
        rc = fk.attend_prefill(q, k, v, out, None, L, 8, 2, 128, 1000, 4, wl.rope_base, check=False)
        torch.cuda.synchronize()
        assert (rc == 0) == ok
        if ok:
            assert (out.float() - want.float()).abs().max() <= 2e-2 * v.float().abs().max()


def test_few_queries_first_call_in_a_capture():
    """A rotary base that no call has had before: nothing is allocated, the table goes into the workspace, and replays read new queries."""
    wl = _wl(hkv=2, hq=8, cap=500, base=54321.0)
    q, k, v = _mk(wl, 500, 3, seed=5)
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, 8, 2, 128, 500, 3)
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        fk.attend_prefill(q, k, v, out, None, L, 8, 2, 128, 500, 3, wl.rope_base, side)
    other = _mk(wl, 500, 3, seed=6)[0]
    for queries in (q.clone(), other, q.clone()):
        q.copy_(queries)
        ws.fill_(255)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        eager, _, _ = _run(q, k, v, wl, 500)
        assert torch.equal(out, eager)
