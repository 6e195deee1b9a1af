"""GPU parity of chunk-wise attention at its start and end: queries rotated by the sum of two angles at the ends of their blocks and at large
positions, results that leave as whole rows from blocks of 1 to 32 queries, in one stream of keys and in halves, and
states merged four parts at a time."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from test_gpu_prefill import TOL_PREFILL, _check, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _wl(hkv, hq, cap):
    return synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=1, batch=1, n_heads=hkv, n_q_heads=hq, window=cap, total_tokens=cap)


def _cut(k, hq, hkv, cur, q_len, size):
    return fk.prefill_cut(binding.layout_for(k), hq, hkv, 128, cur, q_len, size)


@pytest.mark.parametrize("hkv,hq,cur,q_len,halves", [
    (1, 1, 20, 1, 1), (1, 3, 31, 31, 1), (1, 2, 16000, 33, 1),          # fewer rows than the shared table of angles; a long cache
    (1, 8, 70, 1, 2), (1, 8, 95, 31, 2), (1, 6, 96, 33, 2), (2, 14, 64, 63, 2),
])
def test_rows_and_positions(hkv, hq, cur, q_len, halves):
    wl = _wl(hkv, hq, cur)
    _say(f"prefill ends {hkv}/{hq} {cur}/{q_len}")
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)
    _, p = fk.attend_prefill_plan(binding.layout_for(k), hq, hkv, 128, cur, q_len)
    assert _cut(k, hq, hkv, cur, q_len, p.workspace_bytes)[0] == halves
    out, lse, _ = _run(q, k, v, wl, cur)
    assert _check(q, k, v, out, lse, wl, cur) <= TOL_PREFILL


def test_parts_four_at_a_time():
    hkv, hq, cur, q_len = 1, 5, 2300, 35
    wl = _wl(hkv, hq, cur)
    q, k, v = _mk(wl, cur, q_len, seed=3)
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, hq, hkv, 128, cur, q_len)
    states = hq * 2 * 32 * (128 * 4 + 8)
    planned = _cut(k, hq, hkv, cur, q_len, p.workspace_bytes)[1]
    seen = set()
    for parts in range(planned, 0, -1):
        size = p.workspace_bytes - (planned - parts) * states
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        L.workspace, L.workspace_bytes = ws.data_ptr(), size
        out, lse = torch.full_like(q, float("nan")), torch.empty(q.shape[:-1], dtype=torch.float32, device="cuda")
        fk.attend_prefill(q, k, v, out, lse, L, hq, hkv, 128, cur, q_len, wl.rope_base)
        torch.cuda.synchronize()
        seen.add(_cut(k, hq, hkv, cur, q_len, size)[1])
        _say(f"prefill ends, room for {parts} parts")
        assert _check(q, k, v, out, lse, wl, cur, rows=[0, 17, 31, 32, 34]) <= TOL_PREFILL
    assert len({n % 4 for n in seen}) == 4 and max(seen) > 4
