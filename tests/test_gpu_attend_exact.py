"""Decode attention where one row has all the weight: the result is that row of V, to the last bit.  The lanes that share a cache row have to
agree on its score to the last bit for that: each divides what it summed with its own weights by one sum of weights."""
import pytest
import torch

from test_gpu_attend import _mk, _run, _say, _wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("group", [1, 2, 4, 8])
def test_one_row_comes_out_as_it_is(group, d, dtype):
    """A single row, with scores of up to some hundreds; then rows 0, the last and one in between of 2 to 6147, over 150 units of log2 ahead of all
    others in every head, whose weights are thus zero in fp32 (below 2^-149)."""
    hkv, hq = 2, 2 * group
    for cur_len in (1, 2, 65, 700, 6147):
        wl = _wl(d=d, hkv=hkv, hq=hq, cap=cur_len, dtype=dtype)
        for row in sorted({0, cur_len // 2, cur_len - 1}):
            for scale in (0.3, 3.0, 30.0) if cur_len == 1 else (1.0,):
                q, k, v = _mk(wl, cur_len, seed=d + row)
                # query heads along one direction, at their own lengths; that row of K along it too (query at the row's position: no rotation
                # between them), the other rows short
                along = torch.randn(hkv, d, generator=torch.Generator().manual_seed(row + d)).to(q.device)
                lengths = torch.linspace(1.0, 3.0, group, device=q.device)
                q.copy_((along[:, None] * lengths[None, :, None] * scale).reshape(1, 1, hq, d))
                if cur_len > 1:
                    k[..., :cur_len, :] *= 0.25
                    k[0, 0, :, row] = along * (700.0 / d ** 0.5)
                else:
                    k[0, 0, :, row] = along + 0.5 * k[0, 0, :, row]
                out, _, p = _run(q, k, v, wl, cur_len, q_pos=row)
                _say(f"one row {group} {d} {dtype}: {row} of {cur_len}, n_split {p.n_split}")
                assert torch.equal(out[0, 0].view(hkv, group, d), v[0, 0, :, row][:, None].expand(hkv, group, d)), (cur_len, row, scale)
