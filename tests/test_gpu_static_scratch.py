"""Segments at the largest transforms whose workspace of one sky position and one template
the static scratch just holds: the spectra of the plan's own workspace, bit for bit."""
import pytest

import synth
from tests.gpu_util import dev, make_plan, note
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision,interbinning,fits", [
    (524272, 1, 0, True), (524273, 1, 0, False), (524272, 1, 1, True), (524288, 1, 1, False), (262144, 0, 0, True), (262145, 0, 0, False),
    (262144, 0, 1, True), (2048, 1, 0, True), (2048, 0, 0, True)])
def test_largest_segments(torch, n, precision, interbinning, fits):  # noqa: F811
    from paper_1410_3677_amd import fstat as F
    seg = synth.make_segment(n, 2.0, 100.0, 1.0, 7100, [])
    plan = make_plan([seg], precision=precision, interbinning=interbinning)
    nb = synth.nfft_for(n) // 2
    out = [torch.full((2, 2, nb), float("nan"), dtype=torch.float32 if precision else torch.float64, device="cuda")
           for _ in range(2)]
    al, de, fd = dev([0.4, 2.0]), dev([0.1, -0.8]), dev([0.0, -1e-10])
    note(f"n={n} precision={precision} interbinning={interbinning}")
    if not fits:
        with pytest.raises(F.FstatError) as e:
            plan.twoF_spectrum_static(0, al, de, fd, out[1])
        assert e.value.status == F.E_INVAL and "static scratch" in str(e.value)
    else:
        plan.twoF_spectrum(0, al, de, fd, out[0])
        plan.twoF_spectrum_static(0, al, de, fd, out[1])
        torch.cuda.synchronize()
        assert bool(torch.isfinite(out[1]).all()) and torch.equal(out[0], out[1])
    plan.destroy()
