"""Decode attention with two sets of four query heads to a workgroup: numbers of workgroups around the edges of the rule, head sizes, cache types, odd and even
numbers of steps, more steps than between exact angles, ragged lengths; every element against the fp64 oracle, and the same bits as one set to a workgroup."""
import pytest
import torch

from test_gpu_attend import _check, _mk, _run, _run_ragged, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hkv,group,batch,cur_len,dtype", [
    (128, 8, 8, 16, 40, torch.bfloat16),       # 128 workgroups of two sets: one set each
    (128, 3, 8, 43, 40, torch.bfloat16),       # 129 of two sets, two steps
    (128, 8, 8, 17, 97, torch.bfloat16),       # four steps, the last of one row
    (64, 4, 16, 17, 129, torch.bfloat16),      # two workgroups to the same rows; three steps
    (256, 8, 8, 17, 70, torch.bfloat16),       # five steps
    (128, 5, 24, 10, 33, torch.float32),       # three to the same rows; fp32
    (256, 8, 8, 32, 15, torch.float32),        # 256
    (64, 1, 8, 257, 20, torch.bfloat16),       # 257: one set each
    (128, 7, 8, 55, 64, torch.bfloat16),       # 385
    (128, 1, 8, 129, 2200, torch.bfloat16),    # several chunks or more steps than between exact angles
])
def test_two_sets(d, hkv, group, batch, cur_len, dtype):
    wl = _wl(d=d, hkv=hkv, hq=hkv * group, batch=batch, cap=cur_len + 1, dtype=dtype)
    _say(f"two sets d={d} {batch} x {hkv} x {group}, {cur_len} rows, {dtype}")
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    out, lse, p = _run(q, k, v, wl, cur_len)
    assert p.heads_together == 4
    wl3 = _wl(d=d, hkv=hkv, hq=hkv * group, batch=3, cap=cur_len + 1, dtype=dtype)
    for first in (0, batch - 3):               # three sequences at either end by the oracle
        sub = slice(first, first + 3)
        _check(q[:, sub], k[:, sub], v[:, sub], out[:, sub], lse[:, sub], wl3, cur_len)
    if p.n_split == 1:                         # four sequences by themselves, where they have one chunk too: one set to a workgroup
        few, few_lse, p4 = _run(q[:, :4].contiguous(), k[:, :4], v[:, :4], wl, cur_len)
        if p4.n_split == 1 and 4 * hkv * group // 8 <= 128:
            assert torch.equal(few, out[:, :4]) and torch.equal(few_lse, lse[:, :4])


def test_two_sets_ragged_in_chunks():
    """Sequences of 1 to 3000 rows in one call: chunks beyond the short ones are empty in both sets."""
    lens = [3000, 1, 33, 2047, 64, 2999, 500, 1, 1700, 128, 3000, 31, 77, 2500]
    wl = _wl(d=128, hkv=4, hq=32, batch=len(lens), cap=3001)
    q, k, v = _mk(wl, 3000, seed=5)
    for b, n in enumerate(lens):
        k[:, b, :, n:] = float("nan")
        v[:, b, :, n:] = float("nan")
    out, lse, p = _run_ragged(q, k, v, wl, lens)
    assert 128 < len(lens) * 4 * p.n_split <= 256 or len(lens) * 4 * p.n_split > 384
    one = _wl(d=128, hkv=4, hq=32, batch=1, cap=3001)
    for b, n in enumerate(lens):
        _check(q[:, b:b + 1], k[:, b:b + 1], v[:, b:b + 1], out[:, b:b + 1], lse[:, b:b + 1], one, n)
