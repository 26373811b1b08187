"""Host code of the candidate drain on the stand-in HIP runtime (tests/hip_stub.py)."""
import pytest

from tests import hip_stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hip_stub.build(tmp_path_factory.mktemp("stub"))


DRAIN = """
import ctypes, numpy as np
F = H.F
plan = H.plan([4096])
found, flag = 5000, None          # more than one launch drains
u64, u32 = ctypes.POINTER(ctypes.c_ulonglong), ctypes.POINTER(ctypes.c_uint)
def at(args, i, kind):
    return ctypes.cast(ctypes.cast(args[i], ctypes.POINTER(ctypes.c_void_p))[0], kind)
def small(args):                  # head: count, bad, done, two flags
    head = at(args, 4, u64)
    head[0], head[1] = found, 0
def count(args):
    bad = at(args, 8, u32)
    bad[0] = bad[1] = 0
    if flag is not None: bad[flag] = 1
def records(args):
    out, keys, bad, flags = (at(args, i, u32) for i in (6, 7, 8, 9))
    flags[0], flags[1] = bad[0], bad[1]
    if not bad[0]:
        ctypes.memset(out, 0x11, found * 40)
        ctypes.memset(keys, 0x11, found * 24)
H.on.update(k_drain_small=small, k_drain_count=count, k_drain_records=records)
out, keys = np.full(found * 40, 7, np.uint8), np.full(found * 24, 7, np.uint8)
def drain():
    n = ctypes.c_longlong(-1)
    H.launches.clear()
    r = H.lib.fstat_candidates(plan, out.ctypes.data, keys.ctypes.data, found, ctypes.byref(n))
    return r, n.value
assert H.search(plan, 3, 4) == F.OK
"""


@pytest.mark.parametrize("flag", [0, 1])
def test_entries_the_ordering_refused_reach_no_caller(stub, flag):
    """The records' kernel gets the ordering's flags (an entry outside its search, flag 0, has no
    list to form a record from); the call fails before anything is copied to the caller's
    arrays, and keeps the candidates."""
    hip_stub.run(stub, DRAIN + f"""
flag = {flag}
r, n = drain()
assert r == F.E_STATE, r
assert "k_drain_order" in H.names() and "k_drain_reset" not in H.names(), H.names()
assert (out == 7).all() and (keys == 7).all()
flag = None
r, n = drain()
assert r == F.OK and n == found
assert H.names()[-2:] == ["k_drain_records", "k_drain_reset"]
assert (out == 0x11).all() and (keys == 0x11).all()
""")


@pytest.mark.parametrize("failing,use_graph,begun", [
    ("hipStreamBeginCapture", 1, False), ("hipStreamEndCapture", 1, False), ("hipGraphInstantiate", 1, False),
    ("hipGraphLaunch", 1, False), ("k_sky_setup", 1, False), ("k_begin_search", 0, False), ("k_sky_setup", 0, True)])
def test_a_search_that_never_began_is_not_counted(stub, failing, use_graph, begun):
    """The drain's first search index is the device's: a call that fails before its marker
    reaches the device is neither numbered nor recorded, one that fails after it is both."""
    hip_stub.run(stub, f"""
import ctypes
F, failing = H.F, {failing!r}
plan = H.plan([4096], use_graph={use_graph})
device, pending, drained = 0, [], []          # the device's index; launches of the plan's graph; drains
def begin(args):
    global device
    if {use_graph}: pending[:] = [1]
    else: device += 1
def launched(args):
    global device
    device += sum(pending)
def small(args):                              # SmallDrain: nsearch, search0; head: count, bad, done
    a = ctypes.cast(args[0], ctypes.POINTER(ctypes.c_int))
    drained.append((a[0], a[1]))
    head = ctypes.cast(ctypes.cast(args[4], ctypes.POINTER(ctypes.c_void_p))[0], ctypes.POINTER(ctypes.c_ulonglong))
    head[0], head[1] = 0, 1 << 32
H.on.update(k_begin_search=begin, hipGraphLaunch=launched, k_drain_small=small)
assert H.search(plan, 3, 4) == F.OK
ok = H.on.get(failing)
if failing.startswith("hip"):
    H.on[failing] = lambda args: 1
else:                                         # a launch that fails shows at the next look at the errors
    def launch(args):
        if failing == "k_begin_search": pass
        else: (ok or (lambda a: 0))(args)
        H.on["hipGetLastError"] = lambda a: 1
    H.on[failing] = launch
assert H.search(plan, 5, 6) == F.E_DEVICE     # other lists: a graph of its own
H.on.pop("hipGetLastError", None)
if ok: H.on[failing] = ok
else: del H.on[failing]
assert H.search(plan, 7, 8) == F.OK
out, n = ctypes.create_string_buffer(64 * 1024), ctypes.c_longlong()
assert H.lib.fstat_candidates(plan, out, None, 16, ctypes.byref(n)) == F.OK
assert device == {2 + begun}
assert drained == [(device, 0)], (drained, device)
""")
