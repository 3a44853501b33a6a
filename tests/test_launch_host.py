"""Which kernels a plan can be made to launch (no GPU)."""
import ctypes

import pytest

from paper_2201_05278_amd import Propagator, SimwaveError
from paper_2201_05278_amd import _lib as L


def _plan(n, so, scheme="const", dtype="float32", bc=None):
    return Propagator(n, (10.0,) * len(n), so, 1e-4, 20, scheme=scheme, nbl=4, device="cpu", dtype=dtype, bc=bc)


def _tiles(prop, role="forward", extent=7, count=10):
    """Indices that set_launch accepts."""
    out = []
    for tile in range(count):
        try:
            prop.set_launch(tile, extent, role)
            out.append(tile)
            assert (prop.launch(role)["tile"], prop.launch(role)["kind"]) == (tile, "vector")
        except SimwaveError as e:
            assert L.STATUS[e.status] == "SW_ERR_UNSUPPORTED"
    return out


def test_vector_tiles_of_every_scheme_and_role():
    n, free = (40, 44, 48), (("none", "neumann"),) * 3
    assert _tiles(_plan(n, 8)) == list(range(8))
    assert _tiles(_plan(n, 20)) == list(range(7))               # 768 threads with 166 registers each
    assert _tiles(_plan(n, 14), "image_pair") == list(range(7))
    assert _tiles(_plan(n, 8, bc=free)) == list(range(8)) and _tiles(_plan(n, 8, bc=free), "recompute") == []
    assert _tiles(_plan(n, 8, dtype="float64")) == list(range(8)) and _tiles(_plan(n, 8, dtype="float64"), "image") == []
    assert _tiles(_plan(n, 8, "vd_staggered")) == [0, 1, 2, 3, 4]
    assert _tiles(_plan(n, 16, "vd_staggered"), "image") == [0, 1, 3]   # two columns per thread
    assert _tiles(_plan(n, 2, "vd_staggered")) == [] and _tiles(_plan(n, 18, "vd_staggered")) == []
    assert _tiles(_plan(n, 20, "vd_centred")) == [0, 1, 3] and _tiles(_plan(n, 8, "vd_centred"), "recompute") == []


def test_plans_without_an_adjoint_have_no_vector_tiles_for_it():
    n = (40, 44, 48)
    for prop in (_plan(n, 8, "vd_centred"), _plan(n, 8, dtype="float64"), _plan(n, 8, "vd_staggered", bc=(("none", "neumann"),) * 3)):
        assert all(prop.launch(role)["kind"] == "block" for role in ("recompute", "image", "image_pair"))
    assert _plan(n, 8, "vd_staggered").launch("recompute")["kind"] == "vector"


def test_a_launch_is_refused_or_taken_back():
    prop = _plan((40, 44, 48), 8)
    own = prop.launch()
    for bad in ((0, 0), (0, 1 << 20), (0, -3)):
        with pytest.raises(SimwaveError, match="z chunk"):
            prop.set_launch(*bad)
    prop.set_launch(3, 9)
    assert prop.launch() == {"kind": "vector", "tile": 3, "rows": 24, "cols": 64, "zc": 9, "steps": 1}
    assert prop.launch("image")["tile"] != 3 or prop.launch("image")["zc"] != 9
    prop.set_launch()
    assert prop.launch() == own
    prop.set_launch(3, 9)
    prop.set_tiling(8, 8)
    assert prop.launch()["kind"] == "block" and (prop.launch()["rows"], prop.launch()["cols"]) == (8, 64)
    with pytest.raises(SimwaveError, match="tiling of its own"):
        prop.set_launch(3, 9)
    prop.set_tiling()
    assert prop.launch() == own


def test_steps_per_launch_in_2d():
    prop = _plan((60, 80), 8)
    own = prop.launch()
    assert own["kind"] == "steps" and own["steps"] >= 2
    prop.set_launch(1, 3)
    assert prop.launch() == {"kind": "steps", "tile": 1, "rows": 8, "cols": 104, "zc": 0, "steps": 3}
    for bad in ((1, 4), (1, 1), (0, 9), (5, 2)):                # 32 rows hold no output after 4 steps
        with pytest.raises(SimwaveError, match="no such tile"):
            prop.set_launch(*bad)
    prop.set_launch()
    assert prop.launch() == own
    with pytest.raises(SimwaveError, match="no such tile"):
        _plan((60, 80), 8, "vd_staggered").set_launch(1, 3)
    assert _plan((60, 80), 8, "vd_staggered").launch()["kind"] == "block"


def test_an_explicit_2d_tiling_runs_single_steps():
    prop, n = _plan((60, 80), 8), ctypes.c_int64()

    def scratch():
        assert L.lib().sw_plan_scratch(prop._plan, ctypes.byref(n)) == 0
        return n.value

    assert prop.launch()["kind"] == "steps" and scratch() > 0
    prop.set_tiling(zc=16)
    assert (prop.launch()["kind"], prop.launch()["zc"], prop.launch()["steps"]) == ("block", 16, 1) and scratch() == 0
    with pytest.raises(SimwaveError, match="tiling of its own"):
        prop.set_launch(1, 3)
    prop.set_tiling()
    assert prop.launch()["kind"] == "steps" and scratch() > 0


def test_2d_tiles_follow_the_compute_units():
    class Choice(ctypes.Structure):
        _fields_ = [("steps", ctypes.c_int), ("tile", ctypes.c_int)]

    search = getattr(L.lib(), "_ZN2sw14choose_multi2dEiiiii")          # radius, bytes per value, extents, compute units
    search.restype, search.argtypes = Choice, [ctypes.c_int] * 5
    assert search(4, 4, 281, 281, 64).steps < search(4, 4, 281, 281, 256).steps      # tiles queue: less halo per launch


def test_the_benchmark_reports_traffic_of_the_launch_that_was_profiled():
    import bench
    assert bench.profiled_bytes(bench.PROFILED["launch"], 512) == bench.PROFILED["bytes"]
    prop = _plan((512, 512, 512), 8)
    prop.set_launch(bench.PROFILED["launch"]["tile"], bench.PROFILED["launch"]["zc"])
    assert bench.profiled_bytes(prop.launch(), 512) == bench.PROFILED["bytes"]
    prop.set_tiling(24, 8, 74)                  # scalar tiles that move other bytes
    assert bench.profiled_bytes(prop.launch(), 512) is None


def test_threads_share_a_plan():
    """Threads that ask one plan for its tilings (each of them caches occupancies in it) agree with a plan asked alone."""
    from concurrent.futures import ThreadPoolExecutor
    for scheme in ("const", "vd_staggered", "vd_centred"):
        alone, shared = _plan((90, 70, 80), 12, scheme), _plan((90, 70, 80), 12, scheme)
        want = (alone.tiling, alone.launch())
        with ThreadPoolExecutor(8) as pool:
            got = list(pool.map(lambda _: (shared.tiling, shared.launch()), range(64)))
        assert all(g == want for g in got)


@pytest.mark.parametrize("n,so,dtype,kind", [
    ((4010, 4030), 8, "float64", "block"),
    ((4010, 4030), 10, "float64", "block"),         # single steps are 1.2 to 1.35 times as fast
    ((2000, 2000), 10, "float64", "steps"),
    ((1100, 1130), 12, "float64", "block"),
    ((750, 1030), 12, "float64", "steps"),
    ((720, 710), 14, "float64", "block"),
    ((500, 500), 14, "float64", "steps"),
    ((11560, 2510), 10, "float32", "block"),
    ((7460, 2600), 10, "float32", "steps"),
    ((1940, 15280), 12, "float32", "block"),
    ((4500, 3570), 12, "float32", "steps"),
    ((979, 1954), 20, "float32", "block"),
    ((900, 900), 20, "float32", "steps"),
])
def test_2d_grids_that_take_single_steps(n, so, dtype, kind):
    assert _plan(n, so, dtype=dtype).launch()["kind"] == kind
