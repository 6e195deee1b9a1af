"""Decode attention where a KV head has more query heads than are handled together: its workgroups stand in order of units, 8 at a time.
Numbers of chunks below, at and above multiples of 8, two to five parts of a group, one chunk per unit and several."""
import pytest

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,group,batch,cur_len", [(1, 8, 1, 40), (7, 8, 1, 40), (2, 8, 4, 33), (3, 12, 3, 64), (1, 3, 11, 20), (5, 10, 1, 50),
                                                     (1, 8, 1, 3000), (2, 16, 2, 1500), (3, 6, 1, 2000), (1, 20, 3, 700)])
def test_groups_of_many_heads(hkv, group, batch, cur_len):
    wl = _wl(d=128, hkv=hkv, hq=hkv * group, batch=batch, cap=cur_len)
    q, k, v = _mk(wl, cur_len, seed=cur_len + group)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"groups {hkv} x {group}, batch {batch}: {p.heads_together} together, n_split {p.n_split}")
    assert p.heads_together < group
    _check(q, k, v, out, lse, wl, cur_len)
