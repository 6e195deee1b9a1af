"""GPU parity of the near/far form on spans whose leaves' moments go through the workspace, against the fp64 CPU oracle, every element:
windows of 2 and 3 leaves and each count of second parts, tables that repeat and that do not, last blocks of 1 to 4 leaves, the longest
span; many tasks per workgroup, as a workspace of the least size leaves them, against one each; sequences of unlike lengths; a value that
is not finite."""
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import binding, synth

from _util import TOL_BF16
from test_gpu_parity import _check_all_heads, _mk, _run, _say

pytestmark = pytest.mark.gpu


def _workload(span, ratio, **kw):
    args = dict(n_layers=1, batch=1, n_heads=1, head_dim=32, window=span + 4, retain_ratio=ratio, total_tokens=span + 4)
    args.update(kw)
    return synth.small(synth.WORKLOADS["llama2_7b_layer"], **args)


def _kernel(wl):
    L = binding.Layout()
    L.dtype, L.n_layers, L.batch, L.token_capacity, L.stride_token = fk.BF16, 1, 1, wl.window, wl.head_dim
    return fk.compress_kernel(L, 1, wl.head_dim, wl.window, wl.n_sink, wl.retain_ratio)


def _spills(wl):
    assert _kernel(wl) == "k_nearfar (workspace)"


@pytest.mark.parametrize("span,ratio", [
    (14849, 0.5), (15231, 0.5), (14850, 0.6), (16384, 0.9), (13953, 0.75),     # 2 leaves; 117, 119, 117, 128 and 110 of them in all
    (16384, 0.5), (15104, 0.5),                                    # ... with tables that repeat
    (13800, 0.4), (16383, 0.33),                                   # 3 leaves, 10 steps with a second part
    (8705, 0.2), (10300, 0.25), (11787, 0.21), (16384, 0.25),      # 3 leaves, 12 steps; the last with tables that repeat
])
def test_spill_every_element(span, ratio):
    _every_element(span, ratio, "k_nearfar (workspace)")


@pytest.mark.parametrize("span,ratio", [(14801, 0.5), (14848, 0.5), (12800, 0.9), (13312, 0.4), (10237, 0.25), (8704, 0.21)])
def test_longest_spans_without_the_workspace(span, ratio):
    """Both kinds of window with the fewest ring slots, the last span before the workspace is used among them."""
    _every_element(span, ratio, "k_nearfar")


def _every_element(span, ratio, kernel):
    wl = _workload(span, ratio)
    _say(f"spill {span} {ratio}")
    assert _kernel(wl) == kernel
    k, v = _mk(wl, seed=span, capacity=span + 20, cur_len=span + 9)
    k0, v0 = k.cpu().clone(), v.cpu().clone()
    rc, p, tap = _run(k, v, wl, span + 9)
    assert rc == 0 and p.runs == 7
    worst = _check_all_heads(wl, k0, v0, k.cpu(), v.cpu(), tap.cpu(), p, span + 9, TOL_BF16)
    assert worst <= 5e-3                                    # exact entries in 16 bits, as in test_gpu_nearfar


@pytest.mark.parametrize("span,ratio", [(10397, 0.25), (14813, 0.6), (16384, 0.5)])
def test_spill_many_tasks(span, ratio):
    """4 heads in 40 slabs, 160 tasks of 32 channels: with the least workspace a plan names, which holds the moments of some 30
    workgroups, and with a workgroup for each."""
    wl = _workload(span, ratio, n_heads=4, n_layers=20)
    _spills(wl)
    k, v = _mk(wl, seed=7)
    k1, v1 = k.clone(), v.clone()
    L = binding.layout_for(k)
    _, p = fk.plan(L, 4, 32, wl.window, wl.window, wl.n_sink, ratio)
    assert p.workspace_min_bytes > 0
    stream = torch.cuda.current_stream()
    for kk, vv, size in ((k, v, p.workspace_min_bytes), (k1, v1, p.workspace_bytes)):
        ws = torch.full((size,), 0xff, dtype=torch.uint8, device="cuda")        # NaN patterns
        L.workspace, L.workspace_bytes = ws.data_ptr(), size
        assert fk.compress(kk, vv, L, 4, 32, wl.window, wl.window, wl.n_sink, ratio, stream) == 0
        torch.cuda.synchronize()
    assert torch.equal(k[:, :, :, :p.new_len], k1[:, :, :, :p.new_len]) and torch.equal(v[:, :, :, :p.new_len], v1[:, :, :, :p.new_len])
    L.workspace_bytes = p.workspace_min_bytes - 256
    assert fk.compress(k, v, L, 4, 32, wl.window, wl.window, wl.n_sink, ratio, stream, check=False) == -3


def test_spill_tasks_of_one_workgroup():
    """More tasks than compute units: every head alone gives the same bits."""
    heads = 150
    wl = _workload(10300, 0.25, n_heads=heads)
    _spills(wl)
    k, v = _mk(wl, seed=9)
    k0, v0 = k.clone(), v.clone()
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    assert rc == 0
    for h in (0, 77, heads - 1):
        kh, vh = k0[:, :, h:h + 1].clone(), v0[:, :, h:h + 1].clone()
        _run(kh, vh, synth.small(wl, n_heads=1), wl.window, tap=False)
        assert torch.equal(kh[:, :, :, :p.new_len], k[:, :, h:h + 1, :p.new_len])
        assert torch.equal(vh[:, :, :, :p.new_len], v[:, :, h:h + 1, :p.new_len])


def test_spill_ragged():
    wl = _workload(14813, 0.6, batch=3, n_heads=2, n_layers=2)
    _spills(wl)
    lens = [wl.window + 5, wl.window - 1, wl.window]
    k, v = _mk(wl, seed=2, capacity=wl.window + 5, cur_len=wl.window + 5)
    k0, v0 = k.clone(), v.clone()
    L = binding.layout_for(k)
    _, p = fk.plan(L, 2, 32, wl.window, wl.window, wl.n_sink, 0.6)
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    L.workspace, L.workspace_bytes = ws.data_ptr(), ws.numel()
    rc, after = fk.compress_ragged(k, v, L, 2, 32, lens, wl.window, wl.n_sink, 0.6, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert list(after) == [p.new_len + 5, wl.window - 1, p.new_len]
    for b in (0, 2):
        kb, vb = k0[:, b:b + 1].contiguous(), v0[:, b:b + 1].contiguous()
        _run(kb, vb, synth.small(wl, batch=1), lens[b], tap=False)
        n = after[b]
        assert torch.equal(kb[:, 0, :, :n], k[:, b, :, :n]) and torch.equal(vb[:, 0, :, :n], v[:, b, :, :n])
    assert torch.equal(k[:, 1], k0[:, 1]) and torch.equal(v[:, 1], v0[:, 1])


@pytest.mark.parametrize("span,ratio", [(14849, 0.5), (14813, 0.6), (10397, 0.25)])
def test_spill_nan_stays_in_its_channel(span, ratio):
    wl = _workload(span, ratio, head_dim=64)
    _spills(wl)
    k, v = _mk(wl, seed=4)
    clean = k.clone()
    k[0, 0, 0, 4 + 9000, 17] = float("nan")
    rc, p, _ = _run(k, v, wl, wl.window, tap=False)
    _run(clean, v.clone(), wl, wl.window, tap=False)
    got = k[0, 0, 0, 4:p.new_len].float()
    ok = [c for c in range(64) if c != 17]
    assert rc == 0 and not torch.isfinite(got[:, 17]).any()
    assert torch.equal(got[:, ok], clean[0, 0, 0, 4:p.new_len].float()[:, ok])
