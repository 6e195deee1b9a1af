"""Decode attention over values that are infinite or NaN: the channel that holds one takes it, whichever row it is in (the last of the cache, of a chunk of
rows, and the first of the next, whose rows a step of the chunk before may read), and the other channels keep their bits."""
import pytest
import torch

from paper_2505_00570_amd import binding
from test_gpu_attend import _check, _mk, _run, _run_ragged, _say, _wl

pytestmark = pytest.mark.gpu
CHANNEL = 17


@pytest.mark.parametrize("cur_len", [1, 33, 300, 2113])
@pytest.mark.parametrize("d,hkv,group,batch,dtype", [
    (128, 2, 1, 1, torch.bfloat16), (128, 2, 2, 1, torch.bfloat16), (128, 1, 3, 2, torch.bfloat16), (128, 2, 4, 1, torch.bfloat16),
    (64, 2, 1, 2, torch.bfloat16), (64, 1, 4, 1, torch.bfloat16), (256, 1, 2, 1, torch.bfloat16), (256, 1, 4, 2, torch.bfloat16),
    (128, 1, 2, 1, torch.float32), (64, 2, 4, 1, torch.float32), (256, 1, 4, 1, torch.float32),
    (128, 4, 8, 40, torch.bfloat16), (64, 1, 16, 90, torch.float32),        # two sets of four heads to a workgroup
])
def test_values_that_are_not_finite(d, hkv, group, batch, dtype, cur_len):
    wl = _wl(d=d, hkv=hkv, hq=hkv * group, batch=batch, cap=cur_len + 2, dtype=dtype)
    q, k, v = _mk(wl, cur_len, seed=cur_len + d)
    q *= 0.1                                           # weights well above zero for all rows
    clean, _, p = _run(q, k, v, wl, cur_len)
    assert torch.isfinite(clean).all()
    keep = [c for c in range(d) if c != CHANNEL]
    chunk = p.chunk_rows
    for row in sorted({0, cur_len - 1, cur_len - 2, cur_len // 2, chunk - 1, chunk, chunk + 1, cur_len // chunk * chunk} & set(range(cur_len))):
        for value in (float("inf"), float("-inf"), float("nan")):
            _say(f"values that are not finite: d={d} {batch} x {hkv} x {group} {dtype}, row {row} of {cur_len}: {value}")
            v2 = v.clone()
            v2[..., row, CHANNEL] = value
            out, _, _ = _run(q, k, v2, wl, cur_len)
            hit = out[..., CHANNEL].float()
            assert torch.isnan(hit).all() if value != value else (hit == value).all(), (row, value)
            assert torch.equal(out[..., keep], clean[..., keep]), (row, value)


@pytest.mark.parametrize("group", [1, 4])
def test_values_that_are_not_finite_ragged(group):
    lens = [300, 65, 1, 33, 700]
    wl = _wl(hkv=2, hq=2 * group, batch=len(lens), cap=701)
    q, k, v = _mk(wl, 700, seed=2)
    q *= 0.1
    clean, _, _ = _run_ragged(q, k, v, wl, lens)
    keep = [c for c in range(128) if c != CHANNEL]
    v2 = v.clone()
    for b, n in enumerate(lens):
        v2[:, b, :, n - 1, CHANNEL] = float("inf")
        v2[:, b, :, n:] = float("nan")
    out, _, _ = _run_ragged(q, k, v2, wl, lens)
    assert (out[..., CHANNEL].float() == float("inf")).all()
    assert torch.equal(out[..., keep], clean[..., keep])


@pytest.mark.parametrize("group", [1, 4])
def test_rows_beyond_two_gigabytes(group):
    """A cache whose rows lie so far apart that offsets inside a head take all of 32 bits."""
    cur_len, apart = 3000, 1 << 19
    wl = _wl(hkv=1, hq=group, cap=cur_len)
    q, k, v = _mk(wl, cur_len, seed=8)
    far = [torch.empty((cur_len - 1) * apart + 128, dtype=torch.bfloat16, device="cuda").as_strided((1, 1, 1, cur_len, 128), (128, 128, 128, apart, 1))
           for _ in range(2)]
    far[0].copy_(k)
    far[1].copy_(v)
    L = binding.layout_for(far[0])
    assert L.stride_token == apart
    out, lse, _ = _run(q, far[0], far[1], wl, cur_len, layout=L)
    want, want_lse, _ = _run(q, k, v, wl, cur_len)
    _check(q, k, v, out, lse, wl, cur_len)
    assert torch.equal(out, want) and torch.equal(lse, want_lse)
