"""GPU parity of decode attention for one to three KV heads over long caches (chunks that fill a quarter or half of the compute units), with
1, 2 and 4 query heads handled together and 8, 16 and 32 lanes to a row: sums folded in pairs of lane groups."""
import pytest
import torch

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("hkv,group,cur_len", [(1, 1, 8001), (1, 4, 6000), (2, 2, 4097), (3, 4, 5003)])
def test_few_units(hkv, group, cur_len, d, dtype):
    wl = _wl(d=d, hkv=hkv, hq=hkv * group, cap=cur_len, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"few units {hkv} x {group}, {cur_len} rows, {d} {dtype}: n_split {p.n_split}")
    assert p.heads_together == group and 8 < p.n_split * hkv <= 256
    _check(q, k, v, out, lse, wl, cur_len)
