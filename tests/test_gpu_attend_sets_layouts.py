"""Decode attention with two sets of four query heads to a workgroup: caches with other strides and behind pointer tables, a given position of the query,
no rotary embedding, and more workgroups than are there at once."""
import ctypes as C

import pytest
import torch

from paper_2505_00570_amd import binding

from test_gpu_attend import _check, _mk, _run, _wl

pytestmark = pytest.mark.gpu
HKV, HQ, BATCH, CUR = 3, 24, 40, 100                   # 240 workgroups of two sets in two layers, one chunk each


def _case(d=128, dtype=torch.bfloat16, seed=3):
    wl = _wl(d=d, hkv=HKV, hq=HQ, layers=2, batch=BATCH, cap=CUR + 3, dtype=dtype)
    return (wl,) + _mk(wl, CUR, seed=seed)


def _check_some(q, k, v, out, lse, wl, **kw):
    one = _wl(d=wl.head_dim, hkv=HKV, hq=HQ, batch=1, cap=CUR + 3, dtype=wl.dtype)
    for layer, b in ((0, 0), (1, BATCH - 1)):
        at = slice(layer, layer + 1), slice(b, b + 1)
        _check(q[at], k[at], v[at], out[at], lse[at], one, CUR, **kw)


@pytest.mark.parametrize("d,dtype", [(128, torch.bfloat16), (64, torch.float32)])
def test_strided_caches_and_pointer_tables(d, dtype):
    wl, q, k, v = _case(d, dtype)
    want, want_lse, p = _run(q, k, v, wl, CUR)
    assert 128 < 2 * BATCH * HKV * p.n_split <= 256 or 2 * BATCH * HKV * p.n_split > 384
    _check_some(q, k, v, want, want_lse, wl)
    turned = [t.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4) for t in (k, v)]
    padded = []
    for t in (k, v):
        wide = torch.full(t.shape[:4] + (d + 8,), float("nan"), dtype=t.dtype, device="cuda")
        wide[..., :d] = t
        padded.append(wide[..., :d])
    for kk, vv in (turned, padded):
        out, lse, _ = _run(q, kk, vv, wl, CUR)
        assert torch.equal(out, want) and torch.equal(lse, want_lse)
    held = [[t[layer].clone() for layer in range(2)] for t in (k, v)]
    tables = [(C.c_void_p * 2)(*[t.data_ptr() for t in of]) for of in held]
    L = binding.layout_for(k)
    L.pointer_table = 1
    out, lse, _ = _run(q, k, v, wl, CUR, layout=L, kk=tables[0], vv=tables[1])
    assert torch.equal(out, want) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("q_pos", [0, 50, 99, 5000])
def test_given_position(q_pos):
    wl, q, k, v = _case()
    out, lse, _ = _run(q, k, v, wl, CUR, q_pos=q_pos)
    _check_some(q, k, v, out, lse, wl, q_pos=q_pos)


@pytest.mark.parametrize("d", [64, 128, 256])
def test_no_rotary_embedding(d):
    wl, q, k, v = _case(d)
    out, lse, _ = _run(q, k, v, wl, CUR, base=0.0)
    _check_some(q, k, v, out, lse, wl, base=0.0)


@pytest.mark.parametrize("d,group,batch,dtype", [(128, 8, 260, torch.bfloat16), (256, 8, 260, torch.bfloat16), (256, 8, 260, torch.float32), (64, 16, 140, torch.float32)])
def test_more_workgroups_than_three_to_a_compute_unit(d, group, batch, dtype):
    wl = _wl(d=d, hkv=3, hq=3 * group, batch=batch, cap=70, dtype=dtype)
    q, k, v = _mk(wl, 70, seed=9)
    out, lse, p = _run(q, k, v, wl, 70)
    assert batch * 3 * group // 8 * p.n_split > 768
    one = _wl(d=d, hkv=3, hq=3 * group, batch=1, cap=70, dtype=dtype)
    for b in (0, batch - 1):
        at = slice(b, b + 1)
        _check(q[:, at], k[:, at], v[:, at], out[:, at], lse[:, at], one, 70)
