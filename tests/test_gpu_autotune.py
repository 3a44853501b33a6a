"""What the autotuner times and keeps."""
import ctypes
import json

import numpy as np
import pytest
import torch

from paper_2201_05278_amd import Propagator, critical_dt
from paper_2201_05278_amd import _lib as L

pytestmark = pytest.mark.gpu

FREE = (("neumann", "dirichlet"), ("none", "none"), ("none", "none"))


def _prop(n, so, scheme="const", bc=None):
    h = (10.0,) * len(n)
    prop = Propagator(n, h, so, 0.5 * critical_dt(h, so, 3000.0), 20, scheme=scheme, nbl=0, bc=bc)
    rng = np.random.default_rng(0)
    vel = torch.from_numpy(rng.uniform(1500.0, 3000.0, n)).float()
    prop.prepare(vel, None if scheme == "const" else 0.5 * vel, cmax=3000.0)
    return prop


def test_candidates_on_mirror_sides_pay_for_their_ghosts():
    """The tiles that read stored ghosts are timed with the fill that every one of their steps needs: after the call the ghosts
    of the level they read are there."""
    print("case: autotune with mirror sides along z", flush=True)
    prop = _prop((40, 36, 48), 4, bc=FREE)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    fields = [prop.new_field() for _ in range(2)]
    grid = prop.grid_view(fields[0])
    grid.copy_(torch.randn(tuple(grid.shape), generator=g, device="cuda"))
    io = L.FwdIO()
    io.workspace = prop.workspace.data_ptr()
    io.field[0], io.field[1] = fields[0].data_ptr(), fields[1].data_ptr()
    L.check("sw_plan_autotune", L.lib().sw_plan_autotune(prop._plan, ctypes.byref(io), None, None))
    torch.cuda.synchronize()
    lay = prop.layout
    plane = lay.padded[1] * lay.padded[2]
    planes = fields[0].as_strided((40 + 4, 36, 48), (plane, lay.padded[2], 1), lay.origin - 2 * plane)
    assert torch.equal(planes[1], grid[1]) and torch.equal(planes[0], grid[2])          # Neumann: even
    assert torch.equal(planes[42], -grid[38]) and torch.equal(planes[43], -grid[37])    # Dirichlet: odd


def _tuned(prop, cache, **entry):
    """Autotune with a cache file that holds `entry` for the plan."""
    prop.autotune(str(cache))
    text = json.loads(cache.read_text())
    (key,) = text
    known = dict(text[key])
    text[key].update(entry)
    cache.write_text(json.dumps({key: {k: v for k, v in text[key].items() if v is not None}}))
    prop.set_tiling()
    prop.autotune(str(cache))
    return known, json.loads(cache.read_text())[key]


def test_a_tuned_forward_leaves_recompute_and_imaging_to_the_library(tmp_path):
    print("case: gradient launches of a tuned plan", flush=True)
    for scheme in ("const", "vd_staggered"):
        prop = _prop((40, 36, 48), 8, scheme)
        own = {role: prop.launch(role) for role in ("recompute", "image", "image_pair")}
        _tuned(prop, tmp_path / scheme, tx=8, nw=8, zc=20, nt=1, pf=1, wt=0, ts=0, occ=-1, order=0)
        assert (prop.launch()["kind"], prop.launch()["rows"], prop.launch()["zc"]) == ("block", 8, 20)
        for role, was in own.items():
            assert was["kind"] == "vector" and prop.launch(role) == was
        prop.set_tiling(8, 8)                                  # the caller's own choice holds for every role
        assert all(prop.launch(role)["kind"] == "block" for role in own)


def test_a_tuned_2d_plan_keeps_several_steps_per_launch(tmp_path):
    print("case: 2D autotune", flush=True)
    prop = _prop((90, 120), 8)
    own = prop.launch()
    _tuned(prop, tmp_path / "c", zc=12)
    assert own["kind"] == "steps" and prop.launch() == own and prop.tiling["zc"] == 12


def test_cache_entries_of_older_kernels_are_tuned_again(tmp_path):
    print("case: autotune cache of an older library", flush=True)
    prop = _prop((40, 36, 48), 8)
    known, after = _tuned(prop, tmp_path / "c", tx=16, nw=8, zc=5, kernels=None)
    assert after["kernels"] == known["kernels"] and after["zc"] != 5 and prop.tiling["zc"] != 5
