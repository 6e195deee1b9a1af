"""Decode attention with 8 query heads to a KV head on either side of the lines between one and two sets of four heads to a workgroup, which depend on how many
workgroups there are and on whether their steps are odd: every call has the bits of a few of its sequences by themselves, and those are right by the fp64 oracle."""
import pytest
import torch

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workgroups", [130, 256, 258, 384, 386, 512, 514, 640, 642, 768, 770, 896, 898])
@pytest.mark.parametrize("d,dtype", [(128, torch.bfloat16), (64, torch.float32), (256, torch.bfloat16)])
def test_bits_on_either_side(d, dtype, workgroups):
    step = 4096 // d                                   # rows
    for steps in (1, 2, 3, 5, 11):
        cur_len = steps * step - 3
        wl = _wl(d=d, hkv=2, hq=16, batch=workgroups // 2, cap=cur_len, dtype=dtype)
        q, k, v = _mk(wl, cur_len, seed=steps)
        out, lse, p = _run(q, k, v, wl, cur_len)
        if p.n_split != 1:
            continue
        _say(f"lines of sets d={d} {dtype} {workgroups} workgroups of {steps} steps")
        few = _wl(d=d, hkv=2, hq=16, batch=1, cap=cur_len, dtype=dtype)
        _check(q[:, -1:], k[:, -1:], v[:, -1:], out[:, -1:], lse[:, -1:], few, cur_len)
        at = slice(0, 60)                              # 120 workgroups of two sets, or 240 of one: always one set to each
        again, again_lse, p = _run(q[:, at].contiguous(), k[:, at], v[:, at], wl, cur_len)
        if p.n_split == 1:
            assert torch.equal(again, out[:, at]) and torch.equal(again_lse, lse[:, at]), steps
