"""Which kernels a call launches, on the stand-in HIP runtime (tests/hip_stub.py)."""
import pytest

from tests import hip_stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return hip_stub.build(tmp_path_factory.mktemp("stub"))


@pytest.mark.parametrize("precision", [0, 1])
def test_a_plan_with_a_vetter_stays_at_the_full_rate(stub, precision):
    """Windows captured by a search and windows of a spectrum of the same plan come from the
    same transforms, however large the spectrum."""
    hip_stub.run(stub, f"""
import ctypes
F = H.F
plan = H.plan([86164], precision={precision}, use_graph=0)
def decimated(call):
    H.launches.clear()
    assert call(plan, 64, 64) == F.OK
    return any(n.startswith("k_tmpl_a_dec") for n in H.names())
vet = ctypes.c_void_p()
assert H.lib.fstat_vet_create(512, ctypes.byref(vet)) == F.OK
assert decimated(H.search) and decimated(H.spectrum)
assert H.lib.fstat_plan_attach_vetter(plan, vet, 100) == F.OK
assert not decimated(H.search) and not decimated(H.spectrum)
assert H.lib.fstat_plan_attach_vetter(plan, None, 0) == F.OK
assert decimated(H.search) and decimated(H.spectrum)
""")


def test_sky_stages_are_those_of_the_plans_calls(stub):
    """The stage-by-stage entry runs the per-sky kernels that the plan's searches run."""
    hip_stub.run(stub, """
F = H.F
def kernels(plan, call):
    H.launches.clear()
    assert call() == F.OK
    return {n for n in H.names() if "k_spline" in n or "fft_pass" in n or "k_sky_cols" in n or "k_sky_rows" in n}
def stages(plan):
    return kernels(plan, lambda: H.lib.fstat_sky_stages(plan, 0, 0.1, 0.2, None, H.ptr, H.ptr, *[None] * 5))
for n, opts in ((30011, {}), (30011, dict(k_max=65536)), (30011, dict(precision=0)), (86164, dict(interbinning=1)),
                (300007, {}), (300007, dict(interbinning=1))):
    plan = H.plan([n], use_graph=0, **opts)
    want = kernels(plan, lambda: H.search(plan, 64, 64))
    assert want and stages(plan) == want, (n, opts, want)
    assert any("full::" in k for k in want) == (opts == dict(k_max=65536) or n == 300007 and "interbinning" in opts)
""")


# segment, precision, workspace budget in MiB, sky positions and templates a launch that fit it
# at the full rate
@pytest.mark.parametrize("n,precision,mib,skies,templates", [
    (30011, 1, 40, 8, 8), (30011, 1, 64, 8, 32), (30011, 1, 100, 8, 64), (86164, 1, 40, 2, 2), (86164, 1, 100, 4, 8),
    (30011, 0, 40, 4, 4), (30011, 0, 64, 4, 16), (86164, 0, 40, 1, 1), (86164, 0, 100, 2, 4)])
def test_decimated_series_take_no_room_where_launches_are_too_small(stub, n, precision, mib, skies, templates):
    """Budgets under which no launch is large enough to decimate leave the full-rate calls the
    batch sizes that they would have without the decimated series."""
    hip_stub.run(stub, f"""
import ctypes
plan = H.plan([{n}], precision={precision}, workspace_budget_bytes={mib} << 20, use_graph=0)
v = [ctypes.c_int() for _ in range(7)]
assert H.lib.fstat_plan_info(plan, 0, *[ctypes.byref(x) for x in v]) == 0
assert v[3].value >= {templates} and v[4].value >= {skies}, (v[3].value, v[4].value)
assert H.workspace(plan) <= {mib} << 20
assert H.search(plan, 64, 64) == 0 and not any("dec" in k for k in H.names())
""")


@pytest.mark.parametrize("n,precision,templates", [(86164, 0, 4), (120011, 0, 4), (131072, 0, 2), (30011, 0, 16),
                                                   (169509, 1, 4), (200000, 1, 4), (86164, 1, 8), (30011, 1, 32)])
def test_templates_per_launch_on_the_static_scratch(stub, n, precision, templates):
    """One sky position on the static scratch; then the plan's own calls decimate as before."""
    hip_stub.run(stub, f"""
plan = H.plan([{n}], precision={precision}, use_graph=0)
need = H.workspace(plan)
H.launches.clear()
assert H.spectrum(plan, 1, 64, static=True) == 0
a = [k for k in H.names() if k.startswith("k_tmpl_a")]
assert 0 < len(a) <= 64 // {templates} and not any("dec" in k for k in H.names()), a
assert H.workspace(plan) == need
assert H.search(plan, 64, 64) == 0 and any("k_tmpl_a_dec" in k for k in H.names())
""")


@pytest.mark.parametrize("n,precision,opts,arrays,used", [
    (30011, 0, {}, 3, 3), (30011, 1, {}, 4, 3), (30011, 1, dict(k_max=65536), 4, 4), (2048, 1, dict(k_max=4096), 4, 4),
    (300007, 0, dict(interbinning=1), 3, 3)])
def test_per_sky_scratch_is_what_the_stage_uses(stub, n, precision, opts, arrays, used):
    """The per-sky arrays lie between the resampled series and the templates' intermediate,
    with no room beyond them."""
    hip_stub.run(stub, f"""
import ctypes
nb, n, used, size = 5, {n}, {used}, {8 if precision else 16}
M = 1024
while M < n: M *= 2
seen = {{}}
def at(args, i): return ctypes.cast(args[i], ctypes.POINTER(ctypes.c_ulonglong))[0]
H.on.update({{"k_sky_demod": lambda a: seen.__setitem__("z", at(a, 3)),
              "k_sky_rows": lambda a: seen.__setitem__("last", at(a, 0)),                 # in place, behind the odd samples
              "full::k_spline": lambda a: seen.__setitem__("last", at(a, 3)),            # the odd samples, last of all
              "k_tmpl_a": lambda a: seen.__setitem__("tmpl", at(a, 2)),
              "k_tmpl_a_pair": lambda a: seen.__setitem__("tmpl", at(a, 2))}})
plan = H.plan([n], precision={precision}, skies_per_batch=nb, templates_per_launch=256, use_graph=0, **{opts!r})
assert H.search(plan, nb, 64) == 0
one = nb * M * 2 * size                  # an array of pairs
assert seen["last"] + one == seen["z"] + used * one, seen
assert seen["z"] + {arrays} * one <= seen["tmpl"] < seen["z"] + {arrays} * one + 256, (seen, one)
""")


@pytest.mark.parametrize("lengths,opts,nsky,nfdot,first,second", [
    ([2048], dict(templates_per_launch=4096, skies_per_batch=64), 64, 64, "40", "k_tmpl_b_stream<float, 64, 1, 2, 4>"),
    ([4096], dict(templates_per_launch=4096, skies_per_batch=64), 32, 64, "40", "k_tmpl_b_stream<float, 128, 1, 2, 4>"),
    ([5000], dict(templates_per_launch=4096, skies_per_batch=64, interbinning=1), 32, 64, "40", "k_tmpl_b_ib<128, 1, 2>"),
    ([2048, 60001], dict(), 40, 200, "40", "k_tmpl_b_stream<float, 64, 1, 2, 1>"),
    ([30011], dict(templates_per_launch=300, skies_per_batch=7), 17, 67, "160", "k_tmpl_b_stream<float, 256, 1, 2, 4>"),
    ([30011], dict(templates_per_launch=300, skies_per_batch=7, interbinning=1), 17, 67, "80", "k_tmpl_b_ib<256, 1, 2>"),
    ([4097], {}, 16, 64, "80", None), ([12001], {}, 8, 64, "80", None), ([16384], {}, 8, 64, "80", None),
    ([30011], {}, 4, 64, "160", None), ([86164], {}, 2, 32, "320", None), ([131072], {}, 2, 32, "320", None),
    ([150001], {}, 2, 16, "320", None), ([262144], {}, 2, 16, "320", None), ([300007], {}, 2, 8, "640", None),
    ([524288], {}, 2, 8, "640", None), ([262000], dict(interbinning=1), 2, 32, "320", None)])
def test_which_spectra_decimate(stub, lengths, opts, nsky, nfdot, first, second):
    """The grids of the decimated transforms' tests reach every first pass."""
    out = hip_stub.run(stub, f"""
plan = H.plan({lengths!r}, use_graph=0, **{opts!r})
assert H.spectrum(plan, {nsky}, {nfdot}) == 0
print("\\n".join(sorted(set(H.names()))))
""")
    assert f"k_tmpl_a_dec<float, {first}, " in out and (second is None or second in out), out


def test_decimated_first_passes_are_those_that_calls_reach(stub):
    """Over every precision, transform length and share of it that the data fill, calls launch
    a kernel each time, and together every instantiation in the library."""
    import re
    import subprocess
    from paper_1410_3677_amd import fstat as F
    out = hip_stub.run(stub, """
F = H.F
for precision in (0, 1):
    for ib in (0, 1):
        for e in range(12 + ib, 21):
            half = 1 << (e - 1)
            for n in sorted({max(2048, v) for v in (half // 2 + 1, 3 * half // 4, 5 * half // 7, half - 100, half)}):
                plan = H.plan([n], precision=precision, interbinning=ib, nfft=2 * half, templates_per_launch=4096,
                              skies_per_batch=8, use_graph=0)
                assert H.search(plan, 8, 512) == F.OK, (precision, ib, e, n, H.lib.fstat_last_error(plan))
                H.lib.fstat_destroy(plan)
print("\\n".join(sorted(set(H.names()))))
""")
    syms = subprocess.run(["nm", "-DC", "--defined-only", F.LIB_PATH], capture_output=True, text=True, check=True).stdout
    built = set(re.findall(r"\bk_tmpl_a_dec<[^>]*>", syms))
    assert built and built == set(re.findall(r"\bk_tmpl_a_dec<[^>]*>", out))
