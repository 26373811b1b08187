"""The per-sky stage against the oracle over every transform length, at both ends of a
length's range, on irregular delays and on sampling intervals of whole half sidereal days.

Bounds: a double-precision value inherits the demodulation phase's rounding
(phase_conditioning), times a small factor; single-precision ones are those of the full-size
stage test.  The antenna averages are closed forms of the sidereal phase, which n samples
carry to n rate dt radians at 2^-53 relative."""
from __future__ import annotations

import math

import numpy as np
import pytest

import synth
from tests.gpu_util import note
from tests.test_gpu_parity import _stage_errors, phase_conditioning, torch  # noqa: F401

pytestmark = pytest.mark.gpu
RATE = 2 * math.pi / 86164.0905


def _check(torch, seg, al, de, fp64):
    e = _stage_errors(torch, seg, al, de, fp64)
    note(f"n={seg.n} fp64={fp64}: " + ", ".join(f"{k} {v:.1e}" for k, v in e.items()))
    avg = 1e-13 + 8 * seg.n * RATE * seg.dt * 2.0 ** -53
    assert max(e["A"], e["B"], e["C"]) < avg
    series = [e[k] for k in ("za", "zb", "ua", "ub", "zta", "ztb")]
    if fp64:
        assert max(series) < 8 * phase_conditioning(seg) + 1e-13
    else:
        assert max(series[:2]) < 1e-6 and max(series[2:4]) < 2e-6 and max(series[4:]) < 5e-6


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("n", [2048, 2049, 4097, 8192, 16384, 16385, 32768, 60001, 131072, 131073, 262145, 524288])
def test_stages_over_lengths(torch, n, fp64):  # noqa: F811
    _check(torch, synth.make_segment(n, 2.0, 100.0, 1.0, 9000 + n), 0.7 + n % 5, 0.4 - 0.1 * (n % 7), fp64)


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("spread", [40.0, 3000.0])
def test_irregular_delays(torch, spread, fp64):  # noqa: F811
    """Delays that jump from sample to sample: by less and by more than a workgroup's knots."""
    seg = synth.make_segment(5000, 2.0, 100.0, 1.0, 9100)
    seg.r[0] += np.random.default_rng(3).uniform(0.0, spread, seg.n)
    _check(torch, seg, 0.3, 0.2, fp64)


@pytest.mark.parametrize("half_days", [1, 2, 3])
@pytest.mark.parametrize("n", [2500, 2501])
def test_averages_at_whole_half_days(torch, n, half_days):  # noqa: F811
    seg = synth.make_segment(n, half_days * 43082.04525, 100.0, 1.0, 9200 + n)
    e = _stage_errors(torch, seg, 1.1, 0.5, True)
    note(f"n={n} dt={seg.dt}: A {e['A']:.1e} B {e['B']:.1e} C {e['C']:.1e}")
    assert max(e["A"], e["B"], e["C"]) < 1e-13 + 8 * n * RATE * seg.dt * 2.0 ** -53
