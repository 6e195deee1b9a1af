"""Into how many chunks of rows decode attention cuts its work (host arithmetic): counts that fill the compute units, and 64 or 128 where few KV heads
over long caches would have more than half as many again."""
import random

import pytest

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding


def _chunks(units, group, d, cur_len, dtype):
    L = binding.Layout()
    L.dtype, L.n_layers, L.batch, L.token_capacity = dtype, 1, 1, cur_len
    L.stride_token, L.stride_head, L.stride_batch = d, d * cur_len, d * cur_len * units
    return fk.attend_plan(L, units * group, units, d, cur_len)[1].n_split


def _in_whole_steps(n, cur_len, d):
    """What becomes of n chunks when each is of whole steps, two of 2048 / d rows."""
    step = 2 * 2048 // d
    chunk = -(-(-(-cur_len // n)) // step) * step
    return -(-cur_len // chunk)


@pytest.mark.parametrize("units,group,d,cur_len,want", [
    # as many as fill the compute units once.  A quarter or half of that takes longer: 5 of 12 7.2 -> 8.6 us, 16 of 32 8.6 -> 10.1, 2 of 5
    # 7.2 -> 8.5, 10 of 24 7.4 -> 8.6, 40 of 74 12.2 -> 13.8, 7 of 25 7.1 -> 8.0, 8 of 16 7.3 -> 8.2
    (12, 2, 64, 1500, 12), (8, 2, 64, 8000, 32), (24, 2, 128, 300, 5), (6, 2, 128, 1500, 24), (3, 2, 128, 16357, 74), (8, 2, 128, 800, 25),
    (16, 1, 128, 1500, 16), (32, 1, 128, 4096, 8), (8, 4, 128, 6147, 28),
    # few KV heads over long caches: 250 chunks 14.9 us, 63 10.1; 128 10.0, 64 8.2; 250 17.5, 125 15.6
    (1, 4, 128, 8000, 63), (2, 4, 64, 8192, 64), (1, 4, 256, 16000, 125),
])
def test_measured_counts(units, group, d, cur_len, want):
    assert _chunks(units, group, d, cur_len, fk.BF16) == want


def test_counts_fill_the_compute_units_or_are_64_or_128():
    r = random.Random(1)
    capped = 0
    for _ in range(3000):
        units, group, d = r.choice([1, 2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 64, 128, 300]), r.choice([1, 2, 3, 4, 8]), r.choice([64, 128, 256])
        cur_len, dtype = round(64 * 256 ** r.random()), r.choice([fk.BF16, fk.F32])
        workgroups = units * group // (4 if group % 4 == 0 else 2 if group % 2 == 0 else 1)
        fills = [max(1, min(256 * k // workgroups, cur_len // (4096 // d))) for k in (1, 2, 3, 4)]
        allowed = {1, *fills} | {cap for cap in (64, 128) if 2 * fills[0] > 3 * cap}
        got = _chunks(units, group, d, cur_len, dtype)
        assert got in {_in_whole_steps(n, cur_len, d) for n in allowed}, (units, group, d, cur_len, dtype, got)
        capped += got not in {_in_whole_steps(n, cur_len, d) for n in {1, *fills}}
    assert capped > 50
