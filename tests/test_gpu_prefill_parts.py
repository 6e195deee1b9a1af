"""GPU parity of chunk-wise attention where few queries meet many keys: the key range is cut into parts whose states are
merged.  Lengths around the edges of tiles and parts, queries that see nothing of a part's first tile, workspaces that hold
fewer parts than the plan names, and the cos/sin table growing from call to call."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from test_gpu_prefill import TOL_PREFILL, _check, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _wl(hkv, hq, cap, layers=1, batch=1):
    return synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=layers, batch=batch, n_heads=hkv, n_q_heads=hq, window=cap,
                       total_tokens=cap)


@pytest.mark.parametrize("hkv,hq,cur,q_len", [(1, 4, 1024, 1), (1, 4, 1025, 33), (2, 2, 2047, 3), (1, 8, 1500, 40), (1, 1, 4000, 257),
                                              (3, 9, 1312, 64), (1, 4, 900, 700), (2, 8, 5001, 301)])
def test_parts_lengths(hkv, hq, cur, q_len):
    wl = _wl(hkv, hq, cur)
    _say(f"prefill in parts {hkv}/{hq} {cur}/{q_len}")
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)
    out, lse, p = _run(q, k, v, wl, cur)
    rows = sorted({0, 1, q_len // 2, q_len - 2, q_len - 1} & set(range(q_len)))
    w = _check(q, k, v, out, lse, wl, cur, rows=rows if q_len > 40 else None)
    assert w <= TOL_PREFILL


def test_smaller_workspace_runs_in_fewer_parts():
    wl = _wl(1, 4, 2048, layers=2)
    q, k, v = _mk(wl, 2048, 50, seed=8)
    out, lse, p = _run(q, k, v, wl, 2048)
    L = binding.layout_for(k)
    _, whole = fk.attend_prefill_plan(L, 4, 1, 128, 2048, 2048)         # a plan without parts needs less
    least = 2048 * 64 * 8 + 2 * (2 * 1) * 64 * 32 * 128 * 2             # cos/sin, rotated keys, transposed values
    assert p.workspace_bytes > least
    for size in (least, (least + p.workspace_bytes) // 2 // 256 * 256, p.workspace_bytes):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        L.workspace, L.workspace_bytes = ws.data_ptr(), size
        again = torch.full_like(q, float("nan"))
        assert fk.attend_prefill(q, k, v, again, None, L, 4, 1, 128, 2048, 50, wl.rope_base) == 0
        torch.cuda.synchronize()
        assert (again.float() - out.float()).abs().max().item() <= 2 ** -7 * out.float().abs().max().item()
    L.workspace_bytes = least - 256
    assert fk.attend_prefill(q, k, v, again, None, L, 4, 1, 128, 2048, 50, wl.rope_base, check=False) == -3


def test_more_rotary_bases_than_tables():
    """From the 17th table of a device on, calls keep the cos/sin in their own workspace: the same results."""
    wl = _wl(1, 2, 70)
    q, k, v = _mk(wl, 70, 20, seed=3)
    torch.cuda.synchronize()
    fk.shutdown()                                     # the tables of other tests
    for i in range(20):
        out, lse, _ = _run(q, k, v, wl, 70, base=1000.0 + i)
        if i in (0, 17, 19):
            assert _check(q, k, v, out, lse, wl, 70, base=1000.0 + i) <= TOL_PREFILL
    again, _, _ = _run(q, k, v, wl, 70, base=1000.0)
    first, _, _ = _run(q, k, v, wl, 70, base=1019.0)
    assert _check(q, k, v, again, None, wl, 70, base=1000.0) <= TOL_PREFILL and torch.equal(first, out)
    torch.cuda.synchronize()
    fk.shutdown()


def test_cos_sin_table_grows():
    for cur in (100, 5000, 300):
        wl = _wl(1, 2, cur)
        q, k, v = _mk(wl, cur, 20, seed=cur)
        out, lse, _ = _run(q, k, v, wl, cur, base=7777.0)
        assert _check(q, k, v, out, lse, wl, cur, base=7777.0) <= TOL_PREFILL
