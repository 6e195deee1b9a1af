"""GPU parity of decode attention for one and two KV heads over long caches (64 or 128 chunks where the compute units would take more than half as
many again), with 1, 2 and 4 query heads handled together and 8, 16 and 32 lanes to a row: sums folded in pairs of lane groups."""
import pytest
import torch

from test_gpu_attend import _check, _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("hkv,group,cur_len,most", [(1, 1, 8001, 64), (1, 4, 8003, 128), (2, 2, 8097, 64), (2, 4, 7000, 64), (1, 4, 16001, 128)])
def test_few_units(hkv, group, cur_len, most, d, dtype):
    wl = _wl(d=d, hkv=hkv, hq=hkv * group, cap=cur_len, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    out, lse, p = _run(q, k, v, wl, cur_len)
    _say(f"few units {hkv} x {group}, {cur_len} rows, {d} {dtype}: n_split {p.n_split}")
    assert p.heads_together == group
    assert 48 < p.n_split <= most and 3 * p.n_split < 2 * min(256 // hkv, cur_len // (4096 // d))      # far fewer than would fill the compute units
    _check(q, k, v, out, lse, wl, cur_len)
