"""Which of its three ways a chunk-wise call takes, asked for in each test: few queries that are still too many to go as heads of a decode call, through the
kernel that works on tiles of keys, at its edges and with its tables of angles; and few queries on strided caches, in many layers and in little room."""
import ctypes as C

import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding

from test_gpu_prefill import TOL_PREFILL, _check, _mk, _run, _say, _wl
from test_gpu_prefill_few import _check_queries

pytestmark = pytest.mark.gpu
OPERANDS, ROWS, DECODE = "k_attend_prefill (operands)", "k_attend_prefill (rows)", "k_attend_quads"
UNTOUCHED = 0xA5


def _way(k, hq, q_len, cur, size=None):
    L = binding.layout_for(k)
    if size is None:
        size = fk.attend_prefill_plan(L, hq, k.shape[2], 128, cur, q_len)[1].workspace_bytes
    return fk.prefill_kernel(L, hq, k.shape[2], 128, cur, q_len, size), fk.prefill_cut(L, hq, k.shape[2], 128, cur, q_len, size)


@pytest.mark.parametrize("hkv,hq,cur,q_len,cut", [
    (1, 72, 20, 1, (1, 1)),            # one query, fewer rows than the shared table of angles
    (1, 65, 70, 1, (2, 1)),            # ... in halves, the last workgroup with one task
    (1, 72, 1024, 1, (2, 3)),          # ... in parts
    (2, 130, 2047, 1, (2, 4)),
    (2, 144, 33, 2, (2, 1)),           # two tiles, the second of one row
    (1, 22, 33, 3, (2, 1)),
    (1, 2, 70, 33, (1, 1)),            # two blocks, the second of one query
    (10, 20, 700, 33, (1, 3)),         # units in a group of eight and beside it, parts that the first block does not see
    (1, 2, 5000, 40, (1, 10)),
])
def test_few_queries_on_tiles(hkv, hq, cur, q_len, cut):
    wl = _wl(hkv=hkv, hq=hq, cap=cur + 2)
    q, k, v = _mk(wl, cur, q_len, seed=cur + q_len)
    _say(f"few queries on tiles {hkv}/{hq} {cur}/{q_len}")
    assert _way(k, hq, q_len, cur) == (OPERANDS, cut)
    out, lse, _ = _run(q, k, v, wl, cur)
    assert _check(q, k, v, out, lse, wl, cur) <= TOL_PREFILL


def _marked(q, k, v, base, cur):
    """Output and workspace of a call whose workspace is marked throughout; the cos/sin of the cached rows have its first cur * 512 bytes."""
    L = binding.layout_for(k)
    _, p = fk.attend_prefill_plan(L, q.shape[2], k.shape[2], 128, cur, q.shape[3])
    ws = torch.full((p.workspace_bytes,), UNTOUCHED, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out = torch.full_like(q, float("nan"))
    fk.attend_prefill(q, k, v, out, None, L, q.shape[2], k.shape[2], 128, cur, q.shape[3], base)
    torch.cuda.synchronize()
    return out, bool((ws[:cur * 512] == UNTOUCHED).all())


def test_more_rotary_bases_than_tables_on_tiles():
    """From the 17th table of a device on, calls have the cos/sin in their own workspace: the same results."""
    wl = _wl(hkv=1, hq=2, cap=70)
    q, k, v = _mk(wl, 70, 40, seed=3)
    assert _way(k, 2, 40, 70)[0] == OPERANDS
    torch.cuda.synchronize()
    fk.shutdown()                                     # the tables of other tests
    outs = []
    for i in range(20):
        out, kept = _marked(q, k, v, 1000.0 + i, 70)
        assert kept == (i < 16), i
        outs.append(out)
        if i in (0, 15, 16, 19):
            assert _check(q, k, v, out, None, wl, 70, base=1000.0 + i) <= TOL_PREFILL
    for i in (0, 19):
        assert torch.equal(_marked(q, k, v, 1000.0 + i, 70)[0], outs[i])
    fk.shutdown()


def test_cos_sin_table_grows_on_tiles():
    """4096 rows of angles at first; a cache of more gets another table, and a shorter one after it either of them."""
    for cur in (100, 5000, 300):
        wl = _wl(hkv=1, hq=2, cap=cur)
        q, k, v = _mk(wl, cur, 40, seed=cur)
        assert _way(k, 2, 40, cur)[0] == OPERANDS
        out, kept = _marked(q, k, v, 7777.0, cur)
        assert kept
        assert _check(q, k, v, out, None, wl, cur, base=7777.0, rows=[0, 1, 31, 32, 39]) <= TOL_PREFILL


@pytest.mark.parametrize("hkv,group,q_len,cur", [(2, 4, 4, 1000), (1, 1, 64, 300), (1, 8, 5, 8000), (1, 1, 1, 16000), (3, 5, 3, 97)])
def test_few_queries_in_the_least_room(hkv, group, q_len, cur):
    """The states of a call of few queries fit where the operands would: the same cut of the rows, and so the same bits, with the least workspace as with the planned one."""
    hq = hkv * group
    wl = _wl(hkv=hkv, hq=hq, cap=cur)
    q, k, v = _mk(wl, cur, q_len, seed=4)
    want, want_lse, p = _run(q, k, v, wl, cur)
    least = -(-cur * 512 // 256) * 256 + 2 * hkv * -(-cur // 32) * 32 * 256
    assert least <= p.workspace_bytes and _way(k, hq, q_len, cur, least)[0] == DECODE == _way(k, hq, q_len, cur)[0]
    assert fk.prefill_kernel(binding.layout_for(k), hq, hkv, 128, cur, q_len, least - 1) is None
    L = binding.layout_for(k)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), least
    out, lse = torch.full_like(q, float("nan")), torch.full_like(want_lse, float("nan"))
    fk.attend_prefill(q, k, v, out, lse, L, hq, hkv, 128, cur, q_len, wl.rope_base)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and torch.equal(lse, want_lse)


def test_few_queries_strided_caches_and_pointer_tables():
    """Token-major rows, padded rows, a pointer table: the bits of the dense cache."""
    hkv, hq, cur, q_len = 2, 6, 385, 5
    wl = _wl(hkv=hkv, hq=hq, layers=3, batch=2, cap=400)
    q, k, v = _mk(wl, cur, q_len, seed=7)
    assert _way(k, hq, q_len, cur)[0] == DECODE
    want, want_lse, p = _run(q, k, v, wl, cur)
    for layer, b in ((0, 0), (2, 1)):
        _check_queries(*(t.cpu() for t in (q, k, v, want, want_lse)), wl, layer, b, cur)
    turned = [t.permute(0, 1, 3, 2, 4).contiguous().permute(0, 1, 3, 2, 4) for t in (k, v)]
    padded = []
    for t in (k, v):
        wide = torch.full(t.shape[:4] + (136,), float("nan"), dtype=t.dtype, device="cuda")
        wide[..., :128] = t
        padded.append(wide[..., :128])
    held = [[t[layer].clone() for layer in range(3)] for t in (k, v)]
    tables = [(C.c_void_p * 3)(*[t.data_ptr() for t in of]) for of in held]
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    for kk, vv, root in ((*turned, None), (*padded, None), (k, v, tables)):
        L = binding.layout_for(kk)
        L.pointer_table = int(root is not None)
        L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
        assert fk.prefill_kernel(L, hq, hkv, 128, cur, q_len, p.workspace_bytes) == DECODE
        out, lse = torch.full_like(q, float("nan")), torch.full_like(want_lse, float("nan"))
        fk.attend_prefill(q, *(root or (kk, vv)), out, lse, L, hq, hkv, 128, cur, q_len, wl.rope_base)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(lse, want_lse)


@pytest.mark.parametrize("q_len", [1, 2])
def test_few_queries_in_more_layers_than_a_pass_holds(q_len):
    """100 layers, 96 to a pass: the first and last layer of either pass."""
    wl = _wl(hkv=1, hq=2, layers=100, cap=130)
    q, k, v = _mk(wl, 129, q_len, seed=8)
    assert _way(k, 2, q_len, 129)[0] == DECODE
    out, lse, _ = _run(q, k, v, wl, 129)
    q, k, v, out, lse = (t.cpu() for t in (q, k, v, out, lse))
    for layer in (0, 95, 96, 99):
        _check_queries(q, k, v, out, lse, wl, layer, 0, 129)
