"""Drains of few crossings (one launch, sorted in LDS) around the sizes where they hand over
to the general drain: every crossing in key order with its record, for exact counts."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import synth
from tests.gpu_util import dev, gpu_spectrum, make_plan, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    w = synth.workload("tiny")
    nb = synth.nfft_for(w.segments[0].n) // 2
    spec = gpu_spectrum(make_plan([w.segments[0]], precision=0), 0, w.alpha, w.delta, w.fdot, nb, True)
    return w, spec


def _threshold(spec, m):
    v = np.sort(spec.ravel())[::-1]
    return float(0.5 * (v[m - 1] + v[m])) if m else float(v[0] + 1.0)


def _check(w, spec, thr, recs, keys, searches):
    at = np.argwhere(spec > thr)
    want = np.concatenate([np.column_stack([np.full(len(at), s), np.zeros(len(at), int), at]) for s in range(searches)])
    got = np.stack([keys[f] for f in ("search", "segment", "sky", "fdot_idx", "bin")], 1)
    np.testing.assert_array_equal(got, want[: len(got)])
    # the same double-precision kernels up to the store: the last place of 2F (1e-13)
    np.testing.assert_allclose(recs["twoF"], spec[tuple(want[: len(got), 2:].T)], rtol=1e-13, atol=0)
    np.testing.assert_array_equal(recs["alpha"], w.alpha[keys["sky"]])
    np.testing.assert_array_equal(recs["fdot"], w.fdot[keys["fdot_idx"]])
    assert np.all(np.isnan(keys["vet_score"]))


@pytest.mark.parametrize("count", [0, 1, 2, 3, 63, 64, 65, 1025, 4095, 4096, 4097])
def test_exact_counts(case, count):
    w, spec = case
    thr = _threshold(spec, count)
    plan = make_plan([w.segments[0]], precision=0, threshold_2F=thr, candidate_capacity=1 << 16)
    for _ in range(2):   # the second pass finds the counter and the lists reset
        plan.search_batch(0, dev(w.alpha), dev(w.delta), dev(w.fdot))
        recs, keys, n = plan.candidates()
        assert n == count
        keys["search"] -= keys["search"].min() if n else 0
        _check(w, spec, thr, recs, keys, 1)


@pytest.mark.parametrize("searches", [3, 4, 5])
def test_several_searches(case, searches):
    w, spec = case
    thr = _threshold(spec, 500)
    plan = make_plan([w.segments[0]], precision=0, threshold_2F=thr, candidate_capacity=1 << 16)
    for _ in range(searches):
        plan.search_batch(0, dev(w.alpha), dev(w.delta), dev(w.fdot))
    recs, keys, n = plan.candidates()
    note(f"{searches} searches: {n} crossings")
    assert n == 500 * searches
    _check(w, spec, thr, recs, keys, searches)


@pytest.mark.parametrize("count", [300, 5000])
def test_partial_and_single_outputs(case, count):
    from paper_1410_3677_amd import fstat as F
    w, spec = case
    thr = _threshold(spec, count)
    plan = make_plan([w.segments[0]], precision=0, threshold_2F=thr, candidate_capacity=1 << 16)

    def drain(recs, keys, capacity):
        plan.search_batch(0, dev(w.alpha), dev(w.delta), dev(w.fdot))
        n = ctypes.c_int64()
        st = plan.lib.fstat_candidates(plan.handle, recs.ctypes.data if recs is not None else None,
                                       keys.ctypes.data if keys is not None else None, capacity, ctypes.byref(n))
        assert n.value == count
        return st
    full, keys = F.candidate_buffers(count)
    assert drain(full, keys, count) == F.OK
    part, pkeys = F.candidate_buffers(100)
    assert drain(part, pkeys, 100) == F.E_OVERFLOW
    np.testing.assert_array_equal(part, full[:100])
    only, _ = F.candidate_buffers(count)
    assert drain(only, None, count) == F.OK
    np.testing.assert_array_equal(only, full)
    _, only_keys = F.candidate_buffers(count)
    assert drain(None, only_keys, count) == F.OK
    np.testing.assert_array_equal(only_keys["bin"], keys["bin"])
    assert drain(part, pkeys, 0) == F.E_OVERFLOW    # nothing asked for: counted and drained
    assert plan.candidate_count() == 0
