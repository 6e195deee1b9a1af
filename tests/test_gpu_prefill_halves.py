"""GPU parity of chunk-wise attention where a workgroup's waves share out the keys in two halves: one and two key tiles, odd
numbers of tiles, tasks that do not fill a workgroup, queries that see nothing of the second half, halves inside parts, and
scores far larger in one half than in the other."""
import pytest

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from test_gpu_prefill import TOL_PREFILL, _check, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _wl(hkv, hq, cap, layers=1, batch=1):
    return synth.small(synth.WORKLOADS["llama3_8b_128k"], n_layers=layers, batch=batch, n_heads=hkv, n_q_heads=hq, window=cap,
                       total_tokens=cap)


def _cut(k, hq, hkv, cur, q_len):
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, hq, hkv, 128, cur, q_len)
    return fk.prefill_cut(L, hq, hkv, 128, cur, q_len, p.workspace_bytes)


@pytest.mark.parametrize("hkv,hq,cur,q_len,cut", [
    (1, 5, 32, 32, (1, 1)),        # one tile: nothing to share out
    (1, 5, 33, 2, (2, 1)),         # two tiles, the second of one row
    (2, 10, 64, 64, (2, 1)),       # two tiles; the first workgroup's queries see the first alone: its second half is empty
    (1, 7, 95, 40, (2, 1)),        # three tiles, 14 tasks: two of the last workgroup's idle
    (2, 8, 250, 200, (2, 1)),      # eight tiles, causal over nearly all
    (3, 9, 481, 70, (2, 1)),       # sixteen tiles, the last of one row
    (1, 8, 1000, 1000, (2, 1)),    # whole chunk without a history
    (1, 6, 1300, 37, (2, 3)),      # halves inside parts of the key range
])
def test_halves_lengths(hkv, hq, cur, q_len, cut):
    wl = _wl(hkv, hq, cur)
    _say(f"prefill in halves {hkv}/{hq} {cur}/{q_len}")
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)
    assert _cut(k, hq, hkv, cur, q_len) == cut
    out, lse, _ = _run(q, k, v, wl, cur)
    rows = sorted({0, 1, 31, 32, q_len // 2, q_len - 2, q_len - 1} & set(range(q_len)))
    assert _check(q, k, v, out, lse, wl, cur, rows=rows if q_len > 40 else None) <= TOL_PREFILL


@pytest.mark.parametrize("loud", [slice(0, 120), slice(120, None)])
def test_halves_of_unlike_scores(loud):
    wl = _wl(1, 5, 240)
    q, k, v = _mk(wl, 240, 20, seed=5)
    assert _cut(k, 5, 1, 240, 20)[0] == 2
    k[..., loud, :] *= 8
    out, lse, _ = _run(q, k, v, wl, 240)
    # q and k are rounded to 11 bits, which shifts a score by a share of its size and an output by as much: 8 times the usual at
    # most.  A half that joins with the wrong weight is off by the size of the output.
    assert _check(q, k, v, out, lse, wl, 240) <= 8 * TOL_PREFILL
