"""Scores in the keys of a drain: a number for each crossing whose window was kept and scored,
NaN for those beyond patch_capacity and those found after the scoring."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, make_plan, note
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision,interbinning,threshold", [
    (4096, 1, 0, 16.0), (4096, 0, 0, 16.0), (8192, 1, 1, 16.0), (8192, 0, 1, 16.0), (30011, 1, 0, 16.0), (140000, 1, 0, 20.0)])
def test_unscored_crossings_have_no_score(torch, n, precision, interbinning, threshold):  # noqa: F811
    from paper_1410_3677_amd import fstat as F
    al, de = synth.fibonacci_sky(4)
    lists = dev(al), dev(de), dev(synth.spindown_grid(6))
    vet = F.Vetter(512)
    vet.set_params((np.random.default_rng(1).standard_normal(vet.n_params) * 0.02).astype(np.float32))
    plan = make_plan([synth.make_segment(n, 2.0, 100.0, 1.0, 6400)], precision=precision, interbinning=interbinning,
                     threshold_2F=threshold, candidate_capacity=1 << 18)
    plan.attach_vetter(vet, 50)
    plan.search_batch(0, *lists)
    plan.vet_candidates()
    plan.search_batch(0, *lists)
    _, keys, found = plan.candidates()
    s = keys["vet_score"]
    note(f"n={n} precision={precision} interbinning={interbinning}: {found} crossings, {int((~np.isnan(s)).sum())} scored")
    assert found > 200 and int((~np.isnan(s)).sum()) == 50
    assert np.isnan(s[keys["search"] == 1]).all()
    assert ((s[~np.isnan(s)] > 0) & (s[~np.isnan(s)] < 1)).all()
    plan.destroy()
