"""Captured searches on the stand-in HIP runtime (tests/hip_stub.py)."""
import pytest

from tests import hip_stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hip_stub.build(tmp_path_factory.mktemp("stub"))


def test_no_graph_outlives_the_batch_sizes_it_was_captured_with(stub):
    """After the autotuner has chosen other batch sizes a search is captured anew, also where
    the new workspace lies at the old one's address."""
    hip_stub.run(stub, """
import ctypes
F = H.F
plan = H.plan([30011])
def sizes():
    v = [ctypes.c_int() for _ in range(7)]
    assert H.lib.fstat_plan_info(plan, 0, *[ctypes.byref(x) for x in v]) == F.OK
    return v[3].value, v[4].value
def search():
    H.launches.clear()
    assert H.search(plan, 40, 30) == F.OK
    return H.names()
before = sizes()
assert "k_begin_search" in search()
assert "k_begin_search" not in search()          # the graph, replayed
assert H.lib.fstat_autotune(plan, 0, 1.0, None) == F.OK
assert sizes() != before
assert "k_begin_search" in search()
assert "k_begin_search" not in search()
""")
