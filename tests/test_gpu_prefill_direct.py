"""Chunk-wise attention that reads the cached rows as they are (tiles that few workgroups use): single heads and rows against the fp64 oracle, in one
stream of keys and in halves, with parts, around the edges of tiles and of the steps between exact angles, on strided caches; and which calls go so."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding
from oracle import attend_oracle as att

from _util import bf16_ulp, f64
from test_gpu_prefill import TOL_PREFILL, _mk, _say, _wl

pytestmark = pytest.mark.gpu


def _call(q, k, v, wl, cur, root=None, base=None):
    """Output, lse, launches that prepare operands, (halves, parts)."""
    L = binding.layout_for(k)
    if root is not None:
        L.pointer_table = 1
    q_len = q.shape[3]
    _, p = fk.attend_prefill_plan(L, wl.q_heads, wl.n_heads, 128, cur, q_len)
    ws = torch.full((p.workspace_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out = torch.full_like(q, float("nan"))
    lse = torch.full(q.shape[:4], float("nan"), dtype=torch.float32, device="cuda")
    fk.profile_enable(True)
    fk.attend_prefill(q, *(root or (k, v)), out, lse, L, wl.q_heads, wl.n_heads, 128, cur, q_len, wl.rope_base if base is None else base)
    torch.cuda.synchronize()
    launches = fk.profile_read().launches_prepare
    fk.profile_enable(False)
    return out.cpu(), lse.cpu(), launches, fk.prefill_cut(L, wl.q_heads, wl.n_heads, 128, cur, q_len, p.workspace_bytes)


def _check_some(q, k, v, out, lse, wl, cur, rope=True):
    """First and last unit, first and last head of a KV head, rows at the ends of blocks: within the tolerance of all chunk-wise calls."""
    q, k, v = q.cpu(), k.cpu(), v.cpu()
    assert not torch.isnan(out.float()).any() and not torch.isnan(lse).any()
    q_len, group = q.shape[3], wl.q_heads // wl.n_heads
    rows = sorted({0, 1, 31, 32, q_len // 2, q_len - 2, q_len - 1} & set(range(q_len)))
    for layer, b, h in {(0, 0, 0), (0, wl.batch - 1, group - 1), (wl.n_layers - 1, wl.batch - 1, wl.q_heads - 1), (wl.n_layers - 1, 0, wl.q_heads // 2)}:
        kk, vv = f64(k[layer, b, h // group, :cur]), f64(v[layer, b, h // group, :cur])
        vmax = float(np.abs(vv).max())
        for i in rows:
            pos = cur - q_len + i
            ref, rlse = att.attend_decode_head(f64(q[layer, b, h, i]), kk, vv, pos + 1, pos, wl.rope_base, rope)
            over = np.maximum(np.abs(f64(out[layer, b, h, i]) - ref) - 0.5 * bf16_ulp(ref) * 1.001, 0.0) / vmax
            assert over.max() <= TOL_PREFILL, (layer, b, h, i, float(over.max()))
            assert abs(float(lse[layer, b, h, i]) - rlse) <= 2e-2, (layer, b, h, i)


@pytest.mark.parametrize("hkv,hq,layers,batch,cur,q_len,cut", [
    (32, 32, 4, 4, 32, 32, (1, 1)),        # one tile
    (32, 32, 4, 4, 33, 20, (1, 1)),        # two tiles, the second of one row
    (32, 32, 4, 2, 190, 65, (1, 1)),       # an even number of steps, idle waves in every workgroup
    (16, 16, 4, 4, 225, 225, (1, 1)),      # an odd one, tasks that do not see the last steps
    (16, 64, 2, 4, 289, 40, (2, 1)),       # halves of five tiles, of which the second has the last row alone
    (32, 32, 2, 2, 505, 250, (2, 1)),      # halves of eight tiles: one set of angles, the first half's alone for early queries
    (16, 32, 2, 4, 1100, 68, (2, 1)),      # halves of eighteen: three sets
    (32, 32, 1, 1, 2300, 28, (1, 6)),      # parts of the key range
    (8, 32, 1, 4, 3333, 39, (2, 4)),       # halves inside parts
])
def test_direct_lengths(hkv, hq, layers, batch, cur, q_len, cut):
    wl = _wl(hkv=hkv, hq=hq, layers=layers, batch=batch, cap=cur + 3)
    _say(f"prefill from the cached rows {layers} x {batch} x {hkv}/{hq} {cur}/{q_len}")
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)       # (rows beyond cur_len are NaN)
    out, lse, launches, got = _call(q, k, v, wl, cur)
    assert launches == 0 and got == cut
    _check_some(q, k, v, out, lse, wl, cur)


def test_direct_strided_caches_and_no_rope():
    """Token-major rows, a pointer table, a padded row: the bits of the dense cache.  And without the rotary embedding."""
    wl = _wl(hkv=16, hq=64, layers=2, batch=4, cap=400)
    q, k, v = _mk(wl, 385, 40, seed=7)
    out, lse, launches, cut = _call(q, k, v, wl, 385)
    assert launches == 0 and cut[0] == 2
    _check_some(q, k, v, out, lse, wl, 385)
    turned = [t.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4) for t in (k, v)]
    padded = []
    for t in (k, v):
        wide = torch.full(t.shape[:4] + (136,), float("nan"), dtype=t.dtype, device="cuda")
        wide[..., :128] = t
        padded.append(wide[..., :128])
    layers = [[t[layer].clone() for layer in range(2)] for t in (k, v)]
    tables = [(C.c_void_p * 2)(*[t.data_ptr() for t in held]) for held in layers]
    for kk, vv, root in ((*turned, None), (*padded, None), (k, v, tables)):
        again, lse2, launches, _ = _call(q, kk, vv, wl, 385, root=root)
        assert launches == 0
        assert torch.equal(again, out) and torch.equal(lse2, lse)
    out, lse, launches, _ = _call(q, k, v, wl, 385, base=0.0)
    assert launches == 0
    _check_some(q, k, v, out, lse, wl, 385, rope=False)


def test_large_and_infinite_values():
    """A value that no fp16 operand holds, in one channel of one row that every query sees: infinite there, the same bits elsewhere."""
    wl = _wl(hkv=32, hq=32, layers=2, batch=2, cap=505)
    q, k, v = _mk(wl, 505, 250, seed=9)
    q *= 0.1
    clean, _, launches, _ = _call(q, k, v, wl, 505)
    assert launches == 0
    keep = [c for c in range(128) if c != 17]
    for row in (0, 100, 250):
        for value in (float("inf"), -1e5):
            loud = v.clone()
            loud[1, 1, 5, row, 17] = value
            out, _, _, _ = _call(q, k, loud, wl, 505)
            want = torch.full((250,), float("inf") if value > 0 else float("-inf"), dtype=out.dtype)
            assert torch.equal(out[1, 1, 5, :, 17], want)
            assert torch.equal(out[..., keep], clean[..., keep])


@pytest.mark.parametrize("hkv,hq,layers,cur,q_len", [(8, 32, 1, 5001, 301), (8, 32, 1, 1000, 1000), (1, 8, 1, 500, 64)])
def test_tiles_of_many_workgroups_have_operands(hkv, hq, layers, cur, q_len):
    wl = _wl(hkv=hkv, hq=hq, layers=layers, cap=cur)
    q, k, v = _mk(wl, cur, q_len, seed=1)
    out, lse, launches, _ = _call(q, k, v, wl, cur)
    assert launches == 1
    _check_some(q, k, v, out, lse, wl, cur)
