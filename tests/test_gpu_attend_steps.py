"""Decode attention: odd and even numbers of loop steps in a chunk, around the count from which a surplus step is left in, for one
chunk and for several, and for lane groups of 8, 16 and 32 lanes, whose sums are folded by different lane swaps."""
import pytest
import torch

import paper_2505_00570_amd as fk

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("steps", [1, 3, 4, 23, 24, 25])
def test_one_chunk(d, steps, dtype):
    """A cache of so many sequences that each is one chunk; the last step's rows but one are past the end."""
    rows = {64: 64, 128: 32, 256: 16}[d]                    # of a step
    wl = _wl(d=d, hkv=4, hq=8, batch=256, cap=rows * steps, dtype=dtype)
    cur_len = rows * (steps - 1) + 1
    q, k, v = _mk(wl, cur_len, seed=steps)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"steps {steps} d {d}: n_split {p.n_split} chunk {p.chunk_rows}")
    assert p.n_split == 1 and p.chunk_rows == rows * steps
    for b in (0, 255):
        s = slice(b, b + 1)
        sub = _wl(d=d, hkv=4, hq=8, batch=1, cap=rows * steps, dtype=dtype)
        _check(q[:, s], k[:, s], v[:, s], out[:, s], lse[:, s], sub, cur_len)


@pytest.mark.parametrize("cur_len", [6147, 6144, 6145, 5376, 800])
def test_several_chunks(cur_len):
    wl = _wl(d=128, hkv=8, hq=32, cap=cur_len)
    q, k, v = _mk(wl, cur_len, seed=cur_len)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"rows {cur_len}: n_split {p.n_split} chunk {p.chunk_rows}")
    assert p.n_split > 1
    _check(q, k, v, out, lse, wl, cur_len)


def test_ragged_lengths_inside_a_chunk_of_odd_steps():
    """Sequences that end after an even, an odd and no step of their last chunk."""
    wl = _wl(d=128, hkv=8, hq=32, batch=4, cap=1536)
    lens = [1536, 1, 700, 1441]
    q, k, v = _mk(wl, 1536, seed=9)
    from paper_2505_00570_amd import binding
    L = binding.layout_for(k)
    _, p = fk.attend_plan(L, 32, 8, 128, 1536)
    ws = torch.empty(max(p.workspace_bytes, 256), dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), p.workspace_bytes
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    fk.attend_decode_ragged(q, k, v, out, lse, L, 32, 8, 128, torch.tensor(lens, dtype=torch.int32, device="cuda"), 1536, wl.rope_base)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        s = slice(b, b + 1)
        _check(q[:, s], k[:, s], v[:, s], out[:, s], lse[:, s], _wl(d=128, hkv=8, hq=32, batch=1, cap=1536), n)
