"""Decimated template transforms of short segments (first passes of 40 points, rows that do not
fill a wavefront's unit of four), interbinned candidates and irregular delays, with batches
large enough that launches of 2^23 points decimate; each test shows that the route was taken
by the last bits, which differ from the full rate's."""
import numpy as np
import pytest

import synth
from oracle import fstat_oracle as ora
from tests.gpu_util import dev, make_plan, note, rel_err_floor
from tests.test_gpu_decimated import HUGE, TOL, _condition, _grid, _segment, _spectra, torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu
LARGE = dict(templates_per_launch=4096, skies_per_batch=64)


def _against_oracle_and_full_rate(torch, plan, seg, al, de, fd, nfft, ib, full_form, k_min, k_max, decimates=True):
    got = _spectra(torch, plan, al, de, fd, k_max - k_min)
    assert bool(torch.isfinite(got).all())
    ref = _spectra(torch, plan, al, de, np.append(fd, HUGE), k_max - k_min)[:, :-1]
    assert torch.equal(got, ref) != decimates        # the route
    far = float(((got - ref).abs() / ref.clamp(min=4.0)).max())
    two_f = ora.template_two_f_interbin if ib else ora.template_two_f
    err = 0.0
    for i, s in ((0, 0), (len(al) - 1, len(fd) - 1)):
        sky = ora.sky_stage(seg, float(al[i]), float(de[i]), nfft)
        want = two_f(seg, sky, float(fd[s]), nfft, k_min, k_max, bool(full_form))
        err = max(err, rel_err_floor(got[i, s].double().cpu().numpy(), want))
    kappa = _condition(seg, al, de, full_form)
    note(f"n={seg.n}: against the full rate {far:.2e}, against the oracle {err:.2e}, condition {kappa:.1f}")
    return far / kappa, err / kappa


@pytest.mark.parametrize("n,ib,full_form,k_min,k_max", [
    (2048, 0, 0, 0, -1), (2049, 0, 0, 0, -1), (4096, 0, 1, 0, -1), (2500, 0, 0, 3, 2999), (3001, 0, 0, 1, 4093),
    (4300, 1, 0, 0, -1), (8100, 1, 0, 0, -1), (8192, 1, 0, 0, -1), (5003, 1, 0, 7, 8100)])
def test_short_spectra_match_oracle_and_full_rate(torch, n, ib, full_form, k_min, k_max):  # noqa: F811
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    al, de, fd = _grid(n, nfft >> ib)
    k_max = nfft // 2 if k_max < 0 else k_max
    plan = make_plan([seg], interbinning=ib, form=full_form, k_min=k_min, k_max=k_max, **LARGE)
    # 8192 samples fill their interbinned transform: no room for the filter's tails
    far, err = _against_oracle_and_full_rate(torch, plan, seg, al, de, fd, nfft, ib, full_form, k_min, k_max, n < 8192)
    assert far < TOL and err < 2 * TOL               # the bounds of test_gpu_decimated.py


@pytest.mark.parametrize("ib", [0, 1])
def test_short_segment_of_a_ragged_plan(torch, ib):  # noqa: F811
    """A short segment beside a long one takes 4096 templates a launch, more sky positions than
    one batch: its candidates are its spectra's crossings."""
    segs = [_segment(5000 if ib else 2048), _segment(60001)]
    nfft = synth.nfft_for(segs[0].n)
    al, de = synth.fibonacci_sky(40)
    fd = synth.spindown_grid(200)
    plan = make_plan(segs, interbinning=ib, threshold_2F=20.0)
    spec = _spectra(torch, plan, al, de, fd, nfft // 2)
    ref = _spectra(torch, plan, al, de, np.append(fd, HUGE), nfft // 2)[:, :-1]
    far = float(((spec - ref).abs() / ref.clamp(min=4.0)).max())
    assert not torch.equal(spec, ref) and far < TOL
    plan.search_batch(0, dev(al), dev(de), dev(fd))
    _, keys, _ = plan.candidates()
    got = {tuple(r) for r in np.stack([keys["sky"], keys["fdot_idx"], keys["bin"]], 1)}
    want = {tuple(r) for r in torch.nonzero(spec > 20.0).cpu().numpy()}
    near = int(((spec - 20.0).abs() < 20.0 * TOL).sum())
    note(f"interbinning={ib}: {len(got)} crossings, {len(got ^ want)} differ, {near} near the threshold, {far:.2e}")
    assert len(want) > 1000 and len(got ^ want) <= near


@pytest.mark.parametrize("ib", [0, 1])
def test_candidates_of_uneven_launches(torch, ib):  # noqa: F811
    """Launches of 300 templates that end within a sky batch of seven."""
    n = 30011
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    al, de = synth.fibonacci_sky(17)
    fd = synth.spindown_grid(67)
    opts = dict(interbinning=ib, templates_per_launch=300, skies_per_batch=7)
    spec = _spectra(torch, make_plan([seg], **opts), al, de, fd, nfft // 2)
    want = {tuple(r) for r in torch.nonzero(spec > 20.0).cpu().numpy()}
    near = int(((spec - 20.0).abs() < 20.0 * TOL).sum())
    found = {}
    for fds in (fd, np.append(fd, HUGE)):
        plan = make_plan([seg], threshold_2F=20.0, **opts)
        plan.search_batch(0, dev(al), dev(de), dev(fds))
        recs, keys, _ = plan.candidates()
        m = keys["fdot_idx"] < len(fd)
        got = {tuple(k): f for k, f in zip(np.stack([keys["sky"], keys["fdot_idx"], keys["bin"]], 1)[m], recs["twoF"][m])}
        found[len(fds)] = got
        note(f"interbinning={ib}, {len(fds)} spindowns: {len(got)} crossings, {len(got.keys() ^ want)} differ, {near} near")
        assert len(want) > 1000 and len(got.keys() ^ want) <= near
    both = found[67].keys() & found[68].keys()
    assert any(found[67][k] != found[68][k] for k in both)          # two routes
    assert all(found[67][k] == float(spec[k]) for k in found[67])   # one route: the spectrum's bits


@pytest.mark.parametrize("n,k_min,k_max", [(2048, 0, 0), (2049, 1, 4090), (4096, 5, 3001)])
def test_rows_of_short_spectra_taken_in_turn(torch, n, k_min, k_max):  # noqa: F811
    """Full-rate launches of 2^23 points and more store four rows' bins together: 2F of the
    same templates one launch each."""
    seg = _segment(n)
    nfft = synth.nfft_for(n)
    nbins = (k_max or nfft // 2) - k_min
    al, de, fd = _grid(n, nfft)
    fd = np.append(fd, HUGE)
    many = _spectra(torch, make_plan([seg], k_min=k_min, k_max=k_max, **LARGE), al, de, fd, nbins)
    one = _spectra(torch, make_plan([seg], k_min=k_min, k_max=k_max, templates_per_launch=1, use_graph=0), al[:3], de[:3],
                   fd, nbins)
    far = float(((many[:3] - one).abs() / one.clamp(min=4.0)).max())
    note(f"n={n} bins [{k_min}, {k_max or nfft // 2}): {far:.2e}")
    assert bool(torch.isfinite(many).all()) and far < TOL


@pytest.mark.parametrize("spread", [40.0, 3000.0])
def test_irregular_delays(torch, spread):  # noqa: F811
    """Delays that jump from sample to sample, by less and by more than the spline's tile.
    The stage is right to 5e-6 of the series' largest value (4.5 of its rms), a bin's
    amplitude so to 2.3e-5 of the noise's, and 2F (floor: the noise's mean) to twice that."""
    seg = _segment(5000)
    seg.r[0] += np.random.default_rng(3).uniform(0.0, spread, seg.n)
    nfft = synth.nfft_for(seg.n)
    al, de, fd = _grid(seg.n, nfft)
    plan = make_plan([seg])
    far, err = _against_oracle_and_full_rate(torch, plan, seg, al, de, fd, nfft, 0, 0, 0, nfft // 2)
    assert max(far, err) < 5e-5
