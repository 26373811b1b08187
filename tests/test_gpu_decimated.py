"""Decimated template transforms (mixed precision, bins below nfft/2): against the oracle
and against the full-rate transforms of the same templates, which a call takes when one of
its spindowns sweeps further than the decimation filter's margin."""
from __future__ import annotations

import math

import numpy as np
import pytest

import synth
from oracle import fstat_oracle as ora
from tests.gpu_util import dev, make_plan, note, rel_err_floor

pytestmark = pytest.mark.gpu

# Bound: the transforms round about twenty times at 2^-24 relative to the spectrum's rms
# (5e-7 of a bin's amplitude, times 4.5 for the extreme of 1e6 bins), doubled in 2F; the
# filter adds at most 5e-8 of the rms.  The full form divides by A B - C^2, which multiplies
# both by 1 / (1 - C^2 / (A B)): one on whole days, up to a thousand on a few hours.
TOL = 1e-5


def _condition(seg, al, de, full_form):
    worst = 1.0
    for a, d in zip(al, de) if full_form else ():
        A, B, C = ora.antenna_averages(*ora.amplitude_modulation(seg.n, seg.dt, float(a), float(d), seg.lat, seg.gamma,
                                                                 seg.phi_r))
        worst = max(worst, 1.0 / (1.0 - C * C / (A * B)))
    return worst


HUGE = 1e-3      # Hz/s: a sweep no margin holds


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch


def _segment(n):
    rng = np.random.default_rng(n)
    return synth.make_segment(n, 2.0, 100.0, 1.0, 8000 + n, synth.draw_injections(rng, 1, 12.0, 12.0))


def _grid(n, points_per_template):
    """Sky and spindown lists just above 2^24 transform points, four spindowns at least."""
    templates = max(8, (1 << 24) // points_per_template)
    nfdot = max(4, min(64, templates // 2))
    nsky = -(-templates // nfdot)
    al, de = synth.fibonacci_sky(nsky)
    return al, de, synth.spindown_grid(nfdot)


def _spectra(torch, plan, al, de, fd, nbins):
    out = torch.full((len(al), len(fd), nbins), float("nan"), dtype=torch.float32, device="cuda")
    plan.twoF_spectrum(0, dev(al), dev(de), dev(fd), out)
    torch.cuda.synchronize()
    return out


# Every first-pass length (5/8 of 64 .. 1024 points) with the fewest and the most nonzero
# first-stage inputs, segments near the ends of their transform's range.
@pytest.mark.parametrize("n,ib,full_form", [
    (2048, 0, 0), (2049, 0, 0), (4096, 0, 1), (4097, 0, 0), (12001, 0, 0), (16384, 0, 0), (30011, 0, 0),
    (86164, 0, 1), (131072, 0, 0), (150001, 0, 0), (262144, 0, 0), (300007, 0, 0), (524288, 0, 0),
    (4300, 1, 0), (8192, 1, 0), (21000, 1, 0), (33000, 1, 0), (60001, 1, 1), (86164, 1, 0), (131072, 1, 0),
    (170000, 1, 0), (262144, 1, 0)])
def test_spectra_match_oracle_and_full_rate(torch, n, ib, full_form):
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    al, de, fd = _grid(n, nfft >> ib)
    plan = make_plan([seg], interbinning=ib, form=full_form)
    note(f"n={n} nfft={nfft} interbinning={ib} grid {len(al)} x {len(fd)}")
    got = _spectra(torch, plan, al, de, fd, nfft // 2)
    assert bool(torch.isfinite(got).all())
    # the same templates at the full rate
    ref = _spectra(torch, plan, al, de, np.append(fd, HUGE), nfft // 2)[:, :-1]
    far = float(((got - ref).abs() / ref.clamp(min=4.0)).max())
    two_f = ora.template_two_f_interbin if ib else ora.template_two_f
    err = 0.0
    for i, s in ((0, 0), (len(al) - 1, len(fd) - 1)):
        sky = ora.sky_stage(seg, float(al[i]), float(de[i]), nfft)
        want = two_f(seg, sky, float(fd[s]), nfft, 0, -1, bool(full_form))
        err = max(err, rel_err_floor(got[i, s].double().cpu().numpy(), want))
    kappa = _condition(seg, al, de, full_form)
    note(f"against the full rate {far:.2e}, against the oracle {err:.2e}, condition {kappa:.1f}")
    assert far < kappa * TOL and err < 2 * kappa * TOL   # the oracle comparison holds the per-sky stage's rounding too


@pytest.mark.parametrize("n,ib,k_min,k_max", [(30011, 0, 1, 32768), (30011, 0, 17, 20001), (86164, 1, 4099, 131072),
                                              (150001, 0, 260000, 262144)])
def test_bin_ranges(torch, n, ib, k_min, k_max):
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    al, de, fd = _grid(n, nfft >> ib)
    whole = _spectra(torch, make_plan([seg], interbinning=ib), al, de, fd, nfft // 2)
    part = _spectra(torch, make_plan([seg], interbinning=ib, k_min=k_min, k_max=k_max), al, de, fd, k_max - k_min)
    far = float(((part - whole[:, :, k_min:k_max]).abs() / part.clamp(min=4.0)).max())
    note(f"n={n} bins [{k_min}, {k_max}): {far:.2e}")
    assert far < TOL


@pytest.mark.parametrize("ib", [0, 1])
def test_candidates_follow_the_spectra(torch, ib):
    """Candidates of a grid whose launches do not divide evenly, and of the same grid with a
    spindown beyond the margin, infinite or not a number (full-rate transforms): those of the
    shared templates are the spectra's crossings."""
    n = 30011
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    al, de, _ = _grid(n, nfft >> ib)
    fd = synth.spindown_grid(67)
    spec = _spectra(torch, make_plan([seg], interbinning=ib), al, de, fd, nfft // 2)
    want = torch.nonzero(spec > 20.0).cpu().numpy()
    near = int(((spec - 20.0).abs() < 20.0 * TOL).sum())
    for bad in (None, HUGE, -HUGE, math.inf, math.nan):
        plan = make_plan([seg], interbinning=ib, threshold_2F=20.0, templates_per_launch=150, skies_per_batch=3)
        plan.search_batch(0, dev(al), dev(de), dev(fd if bad is None else np.append(fd, bad)))
        recs, keys, _ = plan.candidates()
        m = keys["fdot_idx"] < len(fd)
        got = np.stack([keys["sky"][m], keys["fdot_idx"][m], keys["bin"][m]], 1)
        a, b = {tuple(r) for r in got}, {tuple(r) for r in want}
        note(f"interbinning={ib} extra spindown {bad}: {len(a)} crossings, {len(a ^ b)} differ, {near} near the threshold")
        assert len(b) > 1000 and len(a ^ b) <= near and len(a) == len(got)


def test_lattice_templates(torch):
    """Lattice templates (frequency shifts, per-sky spindowns) decimated against the same
    templates of a longer spindown range that no margin holds."""
    from paper_1410_3677_amd import fstat as F
    n = 30011
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    M = synth.lattice_matrix(nfft, 2.0, 100.25, 30, -1e-10, 11)
    lat = F.lattice(M, synth.OBLIQUITY, 100.25)
    sky = F.lattice_sky(lat, 1)
    out = []
    for s_hi in (19, 400):     # 400 steps of 1e-8 in the second matrix's spindown row
        if s_hi == 400:
            M2 = M.copy()
            M2[1, 1] *= 100
        spec = torch.full((len(sky["alpha"]), s_hi + 1, nfft // 2), float("nan"), device="cuda")
        plan = make_plan([seg])
        plan.search_lattice(0, lat if s_hi == 19 else F.lattice(M2, synth.OBLIQUITY, 100.25), sky, 0, s_hi, spectrum=spec)
        torch.cuda.synchronize()
        out.append(spec)
    # spindown index 0 is the same template in both
    far = float(((out[0][:, 0] - out[1][:, 0]).abs() / out[1][:, 0].clamp(min=4.0)).max())
    note(f"{len(sky['alpha'])} sky points: {far:.2e}")
    assert far < TOL
    w1, u = ora.lattice_template(M, 7, float(sky["w_freq"][3]), float(sky["w_spin"][3]), nfft)
    st = ora.sky_stage(seg, float(sky["alpha"][3]), float(sky["delta"][3]), nfft)
    assert rel_err_floor(out[0][3, 7].double().cpu().numpy(), ora.lattice_template_two_f(seg, st, w1, u, nfft)) < 2 * TOL


def test_budget_that_only_full_rate_fits(torch):
    """A workspace budget that one full-rate template fits but not the decimated series
    beside it is still admitted, with the same spectra."""
    seg = _segment(30011)
    nfft = synth.nfft_for(seg.n)
    al, de, fd = _grid(seg.n, nfft)
    import ctypes
    from paper_1410_3677_amd import fstat as F
    need = ctypes.c_size_t()
    one = make_plan([seg], templates_per_launch=1, skies_per_batch=1, workspace_from_torch=False)
    F._check(one.lib.fstat_plan_workspace_size(one.handle, ctypes.byref(need)))
    series = 2 * 2 * 8 * 5 * (6 + (seg.n - 1 + 44) // 8 + 1)   # the two buffers of the decimated series
    plan = make_plan([seg], workspace_budget_bytes=int(need.value) - series // 2)
    note(f"budget {int(need.value) - series // 2}")
    got = _spectra(torch, plan, al, de, fd, nfft // 2)
    ref = _spectra(torch, make_plan([seg]), al, de, fd, nfft // 2)
    assert float(((got - ref).abs() / ref.clamp(min=4.0)).max()) < TOL


@pytest.mark.parametrize("n,k_min,k_max", [(2048, 0, 0), (4097, 3, 8000), (30011, 5, 40006), (150001, 1, 262143)])
def test_spectrum_rows_taken_in_turn(torch, n, k_min, k_max):
    """Full-rate spectra large enough that each lane stores four rows' bins together: the
    same 2F as the same templates one launch each, which store theirs one by one."""
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    nbins = (k_max or nfft // 2) - k_min
    al, de, fd = _grid(n, nfft)
    fd = np.append(fd, HUGE)
    many = _spectra(torch, make_plan([seg], k_min=k_min, k_max=k_max), al, de, fd, nbins)
    one = _spectra(torch, make_plan([seg], k_min=k_min, k_max=k_max, templates_per_launch=1), al, de, fd, nbins)
    far = float(((many - one).abs() / one.clamp(min=4.0)).max())
    note(f"n={n} bins [{k_min}, {k_max or nfft // 2}): {far:.2e}")
    # instantiations may contract differently in the last place of about twenty stages
    assert bool(torch.isfinite(many).all()) and far < TOL
