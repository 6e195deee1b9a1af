"""Tables of rotary angles that chunk-wise calls of few queries keep: as many per device as those of longer chunks, whose table they make ready as well;
beyond that they work in the workspace."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding

from test_gpu_prefill import _mk, _wl
from test_gpu_prefill_few import _check_queries

pytestmark = pytest.mark.gpu
UNTOUCHED = 0xA5


def _call(q, k, v, base, cur, stream=None):
    """(out, lse, workspace) of a call whose workspace is marked throughout."""
    hq, hkv, q_len = q.shape[2], k.shape[2], q.shape[3]
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, hq, hkv, 128, cur, q_len)
    ws = torch.full((p.workspace_bytes,), UNTOUCHED, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out, lse = torch.full_like(q, float("nan")), torch.full(q.shape[:4], float("nan"), dtype=torch.float32, device="cuda")
    fk.attend_prefill(q, k, v, out, lse, L, hq, hkv, 128, cur, q_len, base, stream)
    return out, lse, ws


def test_more_rotary_bases_than_tables_few_queries():
    """From the 17th table of a device on, the angles are in the workspace's first bytes: the same results, and nothing more is allocated."""
    wl = _wl(hkv=1, hq=2, cap=70)
    q, k, v = _mk(wl, 70, 3, seed=3)
    torch.cuda.synchronize()
    fk.shutdown()                                     # the tables of other tests
    results = []
    for i in range(20):
        out, lse, ws = _call(q, k, v, 1000.0 + i, 70)
        torch.cuda.synchronize()
        assert bool((ws[:2048] == UNTOUCHED).all()) == (i < 16), i
        results.append(out)
        if i in (0, 15, 16, 19):
            _check_queries(*(t.cpu() for t in (q, k, v, out, lse)), _wl(hkv=1, hq=2, cap=70, base=1000.0 + i), 0, 0, 70)
    for i in (0, 19):
        assert torch.equal(_call(q, k, v, 1000.0 + i, 70)[0], results[i])
    torch.cuda.synchronize()
    fk.shutdown()


def test_few_queries_make_longer_chunks_ready():
    """A call of few queries ahead of a capture, and in it a long chunk: its cos and sin are kept, as after any other call, and are not worked out by each replay."""
    cur, base = 600, 76543.0
    wl = _wl(hkv=2, hq=8, cap=cur, base=base)
    q, k, v = _mk(wl, cur, 300, seed=5)
    _call(q[:, :, :, -1:].contiguous(), k, v, base, cur)
    torch.cuda.synchronize()
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, 8, 2, 128, cur, 300)
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out = torch.empty_like(q)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        fk.attend_prefill(q, k, v, out, None, L, 8, 2, 128, cur, 300, base, side)
    for _ in range(3):
        ws.fill_(UNTOUCHED)
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert (ws[:cur * 512] == UNTOUCHED).all()
        assert torch.equal(out, _call(q, k, v, base, cur)[0])
        torch.cuda.synchronize()
