"""The per-sky stage of full-rate calls in mixed precision (plans that never decimate, as with
bins up to nfft) against the oracle, as test_gpu_sky_stages.py checks that of decimated ones."""
import numpy as np
import pytest

import synth
from oracle import fstat_oracle as ora
from tests.gpu_util import make_plan, note
from tests.test_gpu_parity import _stages, torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def _check(torch, seg, al, de):
    nfft = synth.nfft_for(seg.n)
    plan = make_plan([seg], k_max=nfft)
    abc, got = _stages(torch, plan, seg, al, de, False)
    other = make_plan([seg])
    _, dec = _stages(torch, other, seg, al, de, False)
    assert not np.array_equal(got[4], dec[4])        # another stage than that of decimated calls
    ref = ora.sky_stage(seg, al, de, nfft)
    want = [ref["za"], ref["zb"], ora.fft_upsample2(ref["za"], nfft), ora.fft_upsample2(ref["zb"], nfft), ref["za_t"],
            ref["zb_t"]]
    err = [float(np.max(np.abs(g - w)) / np.max(np.abs(w))) for g, w in zip(got, want)]
    note(f"n={seg.n}: " + " ".join(f"{e:.1e}" for e in err))
    # the bounds of test_gpu_parity.py's full-size stage test
    assert max(err[:2]) < 1e-6 and max(err[2:4]) < 2e-6 and max(err[4:]) < 5e-6
    plan.destroy()
    other.destroy()


@pytest.mark.parametrize("n", [2048, 2049, 4097, 8192, 16384, 16385, 32768, 60001, 86164, 131072, 131073, 262145, 524288])
def test_stages_over_lengths(torch, n):  # noqa: F811
    _check(torch, synth.make_segment(n, 2.0, 100.0, 1.0, 9000 + n), 0.7 + n % 5, 0.4 - 0.1 * (n % 7))


@pytest.mark.parametrize("spread", [40.0, 3000.0])
def test_irregular_delays(torch, spread):  # noqa: F811
    """Delays that jump from sample to sample: by less and by more than a workgroup's knots."""
    seg = synth.make_segment(5000, 2.0, 100.0, 1.0, 9100)
    seg.r[0] += np.random.default_rng(3).uniform(0.0, spread, seg.n)
    _check(torch, seg, 0.3, 0.2)
