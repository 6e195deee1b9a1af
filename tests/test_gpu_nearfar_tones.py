"""GPU error of the near/far form on channels that are one cosine each, at the retained length and around it: there the rows far from a
result add up in phase instead of cancelling, so that what the far part is rounded to shows.  Against the fp64 CPU oracle, before the
result is rounded; errors are rms over the rms of the channel's span.  White rows beside them."""
import numpy as np
import pytest
import torch

import paper_2505_00570_amd as fk
from paper_2505_00570_amd import synth

from oracle import freqkv_oracle as orc

from _util import f64
from test_gpu_parity import _run, _say

pytestmark = pytest.mark.gpu

OFFSETS = [-60, -25, -16, -12, -9, -7, -5, -4, -3, -2, -1, 0, 1, 2, 3, 4, 5, 7, 9, 12, 16, 25, 40, 60]      # and 8 white channels


def _rows(span, lc):
    j = np.arange(span)
    tones = [np.cos(np.pi * (2 * j + 1) * (lc + o) / (2 * span)) for o in OFFSETS]
    white = np.random.default_rng(span).standard_normal((span, 32 - len(OFFSETS)))
    return torch.from_numpy(np.concatenate([np.stack(tones, 1), white], 1)).to(torch.bfloat16)


def _errors(span, ratio, flags=0):
    """rms error of each channel, of K; V holds the same rows."""
    wl = synth.small(synth.WORKLOADS["llama2_7b_layer"], n_layers=1, batch=1, n_heads=1, head_dim=32, n_sink=0, window=span,
                     retain_ratio=ratio, total_tokens=span)
    lc = min(span, max(1, int(ratio * span + 1e-9)))
    x = _rows(span, lc)
    k, v = (x.to("cuda").reshape(1, 1, 1, span, 32).clone() for _ in range(2))
    rc, p, tap = _run(k, v, wl, span, flags=flags)
    assert rc == 0 and p.retained_len == lc and p.runs == 7 if not flags else p.runs != 7
    ref = orc.compress_span(f64(x), lc)
    got = f64(tap).reshape(2, lc, 32)
    assert np.array_equal(got[0], got[1])
    return np.sqrt(((got[0] - ref) ** 2).mean(0) / (f64(x) ** 2).mean(0))


def _rms(e):
    return float(np.sqrt((e ** 2).mean()))


@pytest.mark.parametrize("span,ratio", [(14850, 0.5), (14813, 0.6), (16384, 0.5), (16384, 0.9), (13800, 0.4), (11787, 0.25), (16384, 0.25), (11260, 0.25),
                                        (10300, 0.21)])
def test_long_spans_are_no_worse_than_the_matrix_form(span, ratio):
    """Spans whose moments go through the workspace took a matrix form of fp16 entries and fp32 sums before there was a near/far form for
    them: no channel may be further off than there."""
    near, matrix = _errors(span, ratio), _errors(span, ratio, fk.FLAG_DENSE)
    t = len(OFFSETS)
    _say(f"tones {span} {ratio}: near/far {_rms(near[:t]):.2e} (max {near[:t].max():.2e}), white {_rms(near[t:]):.2e}; "
         f"matrix {_rms(matrix[:t]):.2e} (max {matrix[:t].max():.2e}), white {_rms(matrix[t:]):.2e}")
    assert (near <= matrix).all()


# rms over the frequencies and over the white channels that the form with a tile at a time reaches at these spans
TILE_AT_A_TIME = [(1008, 0.5, 3.00e-4, 0.955e-4), (1020, 0.5, 3.24e-4, 0.910e-4), (2044, 0.5, 4.01e-4, 0.987e-4), (4092, 0.5, 5.32e-4, 1.042e-4),
                  (6130, 0.5, 5.64e-4, 1.047e-4), (8188, 0.5, 6.00e-4, 1.040e-4), (11260, 0.5, 6.11e-4, 1.036e-4),
                  (1404, 0.25, 1.39e-4, 0.577e-4), (1532, 0.25, 1.51e-4, 0.591e-4), (2048, 0.25, 2.00e-4, 0.662e-4), (4092, 0.25, 2.89e-4, 0.697e-4),
                  (6140, 0.25, 3.54e-4, 0.673e-4), (8188, 0.25, 4.24e-4, 0.687e-4)]


@pytest.mark.parametrize("span,ratio,tones,white", TILE_AT_A_TIME)
def test_units_are_no_worse_than_a_tile_at_a_time(span, ratio, tones, white):
    e, t = _errors(span, ratio), len(OFFSETS)
    _say(f"tones {span} {ratio}: {_rms(e[:t]):.3e} of {tones:.2e} (max {e[:t].max():.2e}), white {_rms(e[t:]):.3e} of {white:.2e}")
    assert _rms(e[:t]) <= tones and _rms(e[t:]) <= white
