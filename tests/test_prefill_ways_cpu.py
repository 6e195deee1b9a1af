"""Which way chunk-wise calls take (host arithmetic): few queries as heads of a decode call, the others on tiles of keys, made by a pass ahead or of the cached rows."""
import random

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding

OPERANDS, ROWS, DECODE = "k_attend_prefill (operands)", "k_attend_prefill (rows)", "k_attend_quads"


def _layout(hkv, cur, layers=1, batch=1, stride=128):
    L = binding.Layout()
    L.dtype, L.n_layers, L.batch, L.token_capacity = fk.BF16, layers, batch, cur
    L.stride_token, L.stride_head = stride, stride * cur
    L.stride_batch, L.stride_layer = stride * cur * hkv, stride * cur * hkv * batch
    return L


def _way(hkv, group, cur, q_len, **kw):
    L = _layout(hkv, cur, **kw)
    size = fk.attend_prefill_plan(L, hkv * group, hkv, 128, cur, q_len)[1].workspace_bytes
    return fk.prefill_kernel(L, hkv * group, hkv, 128, cur, q_len, size)


def test_measured_ways():
    # the shapes that the rules' comments name, as they were timed
    assert _way(32, 1, 4046, 20, batch=4) == _way(32, 1, 1693, 267, layers=2, batch=2) == _way(32, 1, 385, 385, layers=4) == ROWS
    assert _way(32, 1, 794, 794, batch=2) == _way(8, 4, 5082, 121, batch=2) == _way(32, 1, 1631, 17) == ROWS
    assert _way(8, 4, 5001, 301) == _way(8, 4, 1000, 1000) == _way(8, 4, 8192, 4094) == _way(32, 1, 4261, 4261, layers=2) == OPERANDS
    assert _way(8, 4, 888, 888, layers=2, batch=2) == _way(2, 8, 7922, 7) == OPERANDS and _way(8, 2, 6000, 16, layers=4) == ROWS
    assert _way(2, 8, 1500, 8) == _way(8, 4, 1500, 8) == _way(4, 1, 5075, 6, layers=2) == DECODE


def test_up_to_sixteen_queries_go_as_decode_and_more_than_64_never():
    r = random.Random(2)
    ways = set()
    for _ in range(3000):
        hkv, group, layers, batch = r.choice([1, 2, 8, 32]), r.choice([1, 2, 3, 4, 8, 65]), r.choice([1, 1, 4]), r.choice([1, 1, 4])
        cur = round(16 * 1000 ** r.random())
        q_len = min(cur, round(80 ** r.random()))
        way = _way(hkv, group, cur, q_len, layers=layers, batch=batch)
        if group * q_len <= 4:
            assert way == DECODE
        if group * q_len > 64:
            assert way != DECODE
        ways.add(way)
    assert ways == {OPERANDS, ROWS, DECODE}


def test_rows_beyond_31_bits_have_operands():
    """Cached rows are addressed by 31 bits on tiles, by 32 as decode, and a call beyond these is refused."""
    cur = 4000
    assert _way(32, 1, cur, 100, batch=4) == ROWS
    assert _way(32, 1, cur, 100, batch=4, stride=((1 << 30) // (cur + 32)) // 8 * 8) == ROWS
    far = -(-(1 << 30) // (cur + 32)) // 8 * 8 + 8
    assert _way(32, 1, cur, 100, batch=4, stride=far) == OPERANDS
    assert _way(32, 1, cur, 3, batch=4, stride=far) == DECODE
    L = _layout(32, cur, stride=(1 << 31) // (cur + 1024) // 8 * 8 + 8)
    assert fk.attend_prefill_plan(L, 32, 32, 128, cur, 3, check=False)[0] == fk.binding.E_UNSUPPORTED
    assert fk.prefill_kernel(L, 32, 32, 128, cur, 3, 1 << 40) is None


def test_refused_calls_have_no_way():
    L = _layout(8, 1000)
    assert fk.prefill_kernel(L, 32, 8, 128, 1000, 1001, 1 << 40) is None
    assert fk.prefill_kernel(L, 32, 8, 128, 1000, 10, 1000) is None
    assert fk.prefill_kernel(L, 32, 8, 64, 1000, 10, 1 << 40) is None


def test_more_workgroups_than_compute_units_go_as_decode_over_short_caches_only():
    """As decode 38 and 36, 16, 10, 10, 5, 4, 4, 14 and 30 % slower than with operands written first (20.8 us against 15.1 and so on)."""
    assert _way(16, 2, 361, 18, layers=2) == _way(32, 1, 439, 33) == _way(2, 4, 301, 9, layers=4, batch=4) == OPERANDS
    assert _way(8, 1, 213, 40, layers=4) == _way(8, 4, 208, 10, batch=4) == _way(1, 4, 667, 10, layers=4, batch=4) == OPERANDS
    assert _way(8, 2, 152, 20, layers=4) == _way(8, 4, 180, 9, layers=2, batch=2) == OPERANDS
    assert _way(2, 1, 984, 51, layers=2, batch=2) == _way(2, 2, 564, 23, layers=4, batch=2) == OPERANDS
    assert _way(8, 2, 361, 10, layers=2, batch=4) == ROWS            # (as decode 53 % slower)
    # 8, 9, 17, 20 and 17 % faster
    assert _way(16, 2, 92, 11, batch=4) == _way(32, 1, 63, 41) == _way(16, 4, 317, 16) == _way(16, 4, 243, 16) == _way(4, 8, 531, 4, layers=2, batch=2) == DECODE
