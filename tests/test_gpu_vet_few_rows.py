"""Scoring of few patches: the product for few rows forms the sums of the tiled one."""
import numpy as np
import pytest
import torch as _torch  # imported at collection: the first import on a fresh box is slow

from oracle import vet_oracle as vo

pytestmark = pytest.mark.gpu


# one row, the edges of a 16-row tile, and of the range the few-rows product takes
@pytest.mark.parametrize("n", [1, 15, 16, 17, 130, 511, 512])
def test_scores_do_not_depend_on_the_batch(n):
    from paper_1410_3677_amd import fstat as F
    if not _torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    v = F.Vetter(1024)
    v.set_params(vo.init_params(rng).astype(np.float32))
    x = _torch.as_tensor((rng.chisquare(4, size=(600, vo.PATCH)) * rng.uniform(1.0, 6.0, size=(600, 1))).astype(np.float32),
                         device="cuda")
    many = _torch.full((600,), 7.5, device="cuda")
    few = _torch.full((n + 1,), 7.5, device="cuda")
    v.forward(x, many)
    v.forward(x[:n], few[:n])
    # the same products and the same order of sums: the same bits
    assert _torch.equal(few[:n], many[:n]) and float(few[n]) == 7.5
    assert bool(_torch.isfinite(many).all()) and float(many.std()) > 0
