"""The general drain's counting and offsets: one template, many, and either side of one scan tile."""
import numpy as np
import pytest
import torch as _torch  # imported at collection: the first import on a fresh box is slow

import synth
from tests.gpu_util import dev, make_plan, note

pytestmark = pytest.mark.gpu


# entries of one template only; a wavefront's entries from a few templates and from more than the
# eight groups it forms; 4096 templates are one tile of the scan
@pytest.mark.parametrize("ntpl,threshold", [(1, 1.0), (3, 3.0), (4095, 22.0), (4096, 22.0), (4097, 18.0)])
def test_counts_and_order(ntpl, threshold):
    if not _torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 6000 if ntpl < 4 else 2048
    seg = synth.make_segment(n, 2.0, 100.0, 1.0, 41, synth.draw_injections(np.random.default_rng(5), 1, 12.0, 12.0))
    nfft = synth.nfft_for(n)
    al, de = synth.fibonacci_sky(ntpl)
    fd = synth.spindown_grid(1)
    spec = _torch.empty(ntpl, 1, nfft // 2, device="cuda")
    plan = make_plan([seg], threshold_2F=threshold, k_max=nfft // 2)
    plan.twoF_spectrum(0, dev(al), dev(de), dev(fd), spec)
    want = _torch.nonzero(spec > threshold).cpu().numpy()
    plan.search_batch(0, dev(al), dev(de), dev(fd))
    _, keys, _ = plan.candidates()
    got = np.stack([keys[f].astype(np.int64) for f in ("sky", "fdot_idx", "bin")], 1)
    note(f"{ntpl} templates: {len(got)} crossings")
    assert len(want) > 4096          # more than the one-launch drain takes
    assert np.array_equal(got, want)   # key order is the spectrum's order
