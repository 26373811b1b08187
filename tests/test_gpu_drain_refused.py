"""A drain whose crossings belong to no search that the plan knows: a search captured by the
caller and replayed more often than it was called numbers its later crossings beyond the
searches called.  The drain refuses them and leaves the caller's arrays alone."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev, make_plan, note
from tests.test_gpu_decimated import torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threshold,general", [(16.0, False), (8.0, True)])
def test_crossings_of_an_unknown_search(torch, threshold, general):  # noqa: F811
    from paper_1410_3677_amd import fstat as F
    w = synth.workload("tiny")
    al, de, fd = dev(w.alpha), dev(w.delta), dev(w.fdot)
    plan = make_plan(w.segments, threshold_2F=threshold, use_graph=0, candidate_capacity=1 << 18)
    plan.search_batch(0, al, de, fd)
    _, want, n = plan.candidates()
    assert (2 * n > 4096) == general and n > 100
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.search_batch(0, al, de, fd)
    g.replay()
    _, keys, m = plan.candidates()
    assert m == n and np.array_equal(keys["bin"], want["bin"]) and (keys["search"] == 1).all()
    with torch.cuda.graph(g := torch.cuda.CUDAGraph()):
        plan.search_batch(0, al, de, fd)
    g.replay()
    g.replay()
    out = F.candidate_buffers(1 << 18, pinned=True)
    for b in out:
        b.view(np.uint8)[:] = 7
    note(f"threshold {threshold}: {n} crossings a replay, two replays of one call")
    with pytest.raises(F.FstatError) as e:
        plan.candidates(out=out)
    assert e.value.status == F.E_STATE and "outside its search" in str(e.value)
    assert all((b.view(np.uint8) == 7).all() for b in out)
    plan.destroy()
