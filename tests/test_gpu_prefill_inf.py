"""Chunk-wise attention over values that are infinite: a sum that is infinite stays so through the merge of parts of the keys, whichever part it
comes from and however many there are; the other channels keep their bits."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from test_gpu_prefill import _mk, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts", [1, 2, 3, 4, 5, 6])
def test_infinite_values_in_each_part(parts):
    hkv, hq, cur, q_len = 1, 5, 4100, 35                               # planned in 6 parts, of halves
    wl = synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=1, batch=1, n_heads=hkv, n_q_heads=hq, window=cur, total_tokens=cur)
    q, k, v = _mk(wl, cur, q_len, seed=3)
    q *= 0.1                                                              # weights of all rows well above the smallest that fp16 holds
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, hq, hkv, 128, cur, q_len)
    planned = fk.prefill_cut(L, hq, hkv, 128, cur, q_len, p.workspace_bytes)[1]
    size = p.workspace_bytes - max(0, planned - parts) * hq * 2 * 32 * (128 * 4 + 8)
    assert fk.prefill_cut(L, hq, hkv, 128, cur, q_len, size)[1] == parts
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), size

    def run(values):
        out = torch.full_like(q, float("nan"))
        fk.attend_prefill(q, k, values, out, None, L, hq, hkv, 128, cur, q_len, wl.rope_base)
        torch.cuda.synchronize()
        return out

    clean = run(v)
    keep = [c for c in range(128) if c != 17]
    # rows that every query sees, one in each tenth of the keys; infinite as such, and above what an fp16 operand holds
    for row in range(200, cur - q_len, 410):
        for value in (float("inf"), float("-inf"), 1e5):
            v2 = v.clone()
            v2[0, 0, 0, row, 17] = value
            _say(f"infinite values: {parts} parts, row {row}, {value}")
            out = run(v2)
            want = torch.full_like(out[..., 17], float("-inf") if value < 0 else float("inf"))
            assert torch.equal(out[..., 17], want), (row, value)
            assert torch.equal(out[..., keep], clean[..., keep]), (row, value)
