"""Decode attention with one long chunk to a sequence, beyond the steps between exact angles: as many workgroups as go three to a compute unit, and more, which
go by twos; the first and the last sequences against the fp64 oracle."""
import pytest
import torch

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


def _check_ends(d, hkv, group, batch, cur_len, dtype):
    """The first and the last sequence, of a call that has one chunk to each, of more than 64 steps."""
    wl = _wl(d=d, hkv=hkv, hq=hkv * group, batch=batch, cap=cur_len, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"long chunks d={d} {batch} x {hkv} x {group}, {cur_len} rows, {dtype}")
    assert p.heads_together == 4 and p.n_split == 1 and p.chunk_rows > 64 * (4096 // d)
    one = _wl(d=d, hkv=hkv, hq=hkv * group, batch=1, cap=cur_len, dtype=dtype)
    for b in (0, batch - 1):
        sub = slice(b, b + 1)
        _check(q[:, sub], k[:, sub], v[:, sub], out[:, sub], lse[:, sub], one, cur_len)


@pytest.mark.parametrize("d,hkv,batch,cur_len,dtype", [
    (128, 8, 96, 2081, torch.bfloat16),        # 768 workgroups: three to each compute unit; one step beyond the exact angles, its last of a row
    (128, 8, 97, 2049, torch.bfloat16),        # 776: by twos
    (64, 8, 97, 4161, torch.bfloat16),
    (256, 8, 97, 1057, torch.bfloat16),
    (128, 8, 97, 2113, torch.float32),
    (128, 8, 72, 4161, torch.bfloat16),        # exact angles twice
])
def test_long_chunks_of_one_set(d, hkv, batch, cur_len, dtype):
    _check_ends(d, hkv, 4, batch, cur_len, dtype)


@pytest.mark.parametrize("d,hkv,group,batch,cur_len,dtype", [
    (128, 1, 8, 385, 2113, torch.bfloat16),    # two sets of four heads to a workgroup, three steps beyond the exact angles, the last of a row
    (128, 2, 8, 128, 2050, torch.bfloat16),    # 256 workgroups
    (256, 2, 8, 256, 1025, torch.bfloat16),
    (256, 2, 8, 256, 2081, torch.bfloat16),    # exact angles twice
    (64, 2, 8, 200, 4100, torch.bfloat16),
    (64, 1, 16, 200, 4161, torch.float32),     # two workgroups to the same rows
    (256, 1, 8, 400, 1089, torch.float32),
    (128, 1, 8, 400, 2081, torch.float32),
])
def test_long_chunks_of_two_sets(d, hkv, group, batch, cur_len, dtype):
    workgroups = batch * hkv * group // 8
    assert workgroups > 384 or 128 < workgroups <= 256
    _check_ends(d, hkv, group, batch, cur_len, dtype)
