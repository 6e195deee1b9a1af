"""GPU parity of chunk-wise attention where many workgroups see nothing of the later parts of the key range and are not launched: whole
chunks and long ones, with and without halves, in groups of 8 units and beside them, and with each of fewer parts that a smaller
workspace leaves.  Every query block is looked at: one of its first, middle or last rows."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from test_gpu_prefill import TOL_PREFILL, _check, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _wl(hkv, hq, cap, layers=1, batch=1):
    return synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=layers, batch=batch, n_heads=hkv, n_q_heads=hq, window=cap,
                       total_tokens=cap)


@pytest.mark.parametrize("hkv,hq,cur,q_len", [(1, 1, 1600, 1600), (1, 2, 1217, 1217), (2, 6, 1500, 1100), (9, 9, 1100, 1100), (3, 3, 2100, 900),
                                              (10, 10, 700, 33)])
def test_rounds(hkv, hq, cur, q_len):
    wl = _wl(hkv, hq, cur)
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)
    out, lse, p = _run(q, k, v, wl, cur)
    rows = sorted({min(32 * b + (0, 17, 31)[b % 3], q_len - 1) for b in range((q_len + 31) // 32)} | {q_len - 1})
    _say(f"prefill rounds {hkv}/{hq} {cur}/{q_len}")
    assert _check(q, k, v, out, lse, wl, cur, rows=rows) <= TOL_PREFILL
    L = binding.layout_for(k)
    _, plan = fk.attend_prefill_plan(L, hq, hkv, 128, cur, q_len)
    states = hkv * (hq // hkv) * ((q_len + 31) // 32) * 32 * (128 * 4 + 8)          # of a part
    parts = fk.prefill_cut(L, hq, hkv, 128, cur, q_len, plan.workspace_bytes)[1]
    assert parts >= 3
    operands = plan.workspace_bytes - parts * states
    for have in range(parts - 1, -2, -1):
        size = operands + max(have, 0) * states - (256 if have < 0 else 0)           # at last: no room for the operands themselves
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        L.workspace, L.workspace_bytes = ws.data_ptr(), size
        again = torch.full_like(q, float("nan"))
        rc = fk.attend_prefill(q, k, v, again, None, L, hq, hkv, 128, cur, q_len, wl.rope_base, check=False)
        torch.cuda.synchronize()
        assert rc == (0 if have >= 0 else -3)
        if have < 0:
            assert again.isnan().all()
            continue
        assert fk.prefill_cut(L, hq, hkv, 128, cur, q_len, size)[1] <= max(have, 1)
        assert (again.float() - out.float()).abs().max().item() <= 2 ** -7 * out.float().abs().max().item()
