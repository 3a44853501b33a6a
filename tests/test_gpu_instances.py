"""Every vector and multi-step tile, chosen by hand on small ragged grids, bitwise against the scalar single-step kernels
(which the oracle tests pin); and the kernels that the library chooses by itself."""
import time

import numpy as np
import pytest
import torch

from paper_2201_05278_amd import Propagator, SimwaveError, critical_dt, ricker
from paper_2201_05278_amd import _lib as L

pytestmark = pytest.mark.gpu

ODD = (("dirichlet", "neumann"), ("neumann", "dirichlet"), ("none", "neumann"))
H = (10.0, 12.0, 9.0)


def _prop(n, so, steps, nbl=0, scheme="const", dtype="float32", bc=None):
    h = H[:len(n)]
    dt = 0.5 * critical_dt(h, so, 3000.0)
    prop = Propagator(n, h, so, dt, steps, scheme=scheme, nbl=nbl, bc=bc, dtype=dtype)
    mid = [hh * (k - 1) / 2 for k, hh in zip(n, h)]
    prop.set_sources([mid], "linear")
    prop.set_receivers([mid, [0.9 * m for m in mid]], "linear")
    rng = np.random.default_rng(so)
    vel = torch.from_numpy(rng.uniform(1500.0, 3000.0, n)).to(prop.torch_dtype)
    rho = None if scheme == "const" else torch.from_numpy(rng.uniform(1000.0, 2500.0, n)).float()
    prop.prepare(vel, rho, cmax=3000.0)
    return prop, ricker(30.0, dt, steps).reshape(-1, 1).cuda()


def _run(prop, wav, steps=None):
    """Traces and both levels of a run (of `steps` steps) that resumes from noise on the whole grid."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    fields = []
    for _ in range(2):
        f = prop.new_field()
        v = prop.grid_view(f)
        v.copy_(torch.randn(tuple(v.shape), generator=g, device="cuda", dtype=v.dtype))
        fields.append(f)
    res = prop.forward(wav, fields=tuple(fields), step0=1, nsteps_run=steps or prop.nsteps - 1)
    return [res.traces] + [prop.grid_view(f) for f in fields]


def _tiles(prop, extent, roles=("forward",), count=8):
    """Sets each tile that every one of the roles has, in turn."""
    for tile in range(count):
        try:
            for role in roles:
                prop.set_launch(tile, extent, role)
        except SimwaveError as e:
            assert L.STATUS[e.status] == "SW_ERR_UNSUPPORTED"
            continue
        for role in roles:
            assert (prop.launch(role)["kind"], prop.launch(role)["tile"], prop.launch(role)["zc"]) == ("vector", tile, extent)
        yield tile


def _same(a, b):
    assert len(a) == len(b) and float(b[-1].abs().max()) > 0.0
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("so", range(2, 21, 2))
@pytest.mark.parametrize("scheme,dtype", [("const", "float32"), ("const", "float64"), ("vd_staggered", "float32"),
                                          ("vd_centred", "float32")])
def test_every_vector_tile_is_bitwise_the_scalar_tiles(scheme, dtype, so):
    if scheme == "vd_staggered" and so in (2, 18, 20):
        pytest.skip("the staggered scheme has vector tiles from SO4 to SO16")
    # more than two tiles of any extent along x and y, ends inside a vector, uneven chunks
    for bc, n, nbl in ((None, (25, 40, 131), ((2, 0), (9, 4), (5, 7))), (ODD, (27, 45, 133), ((0, 3), (0, 8), (6, 0)))):
        prop, wav = _prop(n, so, 6, nbl, scheme, dtype, bc)
        prop.set_tiling(8, 8)
        ref = _run(prop, wav)
        prop.set_tiling()
        seen = []
        for tile in _tiles(prop, 10):
            print(f"case: {scheme} {dtype} SO{so} vector tile {tile} mirror sides {bc is not None}", flush=True)
            assert _same(_run(prop, wav), ref), (tile, bc)
            seen.append(tile)
        assert len(seen) >= 3


@pytest.mark.parametrize("so", range(2, 21, 2))
@pytest.mark.parametrize("scheme", ["const", "vd_staggered"])
def test_every_vector_tile_of_a_gradient_is_bitwise_the_scalar_tiles(scheme, so):
    if scheme == "vd_staggered" and so in (2, 18, 20):
        pytest.skip("the staggered scheme has vector tiles from SO4 to SO16")
    prop, wav = _prop((25, 40, 131), so, 9, ((2, 0), (9, 4), (5, 7)), scheme)
    roles, every = ("recompute", "image", "image_pair"), 4           # segments of 4, 4 and 1 steps

    def gradient():
        fw = prop.forward(wav, checkpoint_every=every)
        out = prop.adjoint(wav, fw.traces, fw.ckpt, every)
        return [out[0].clone()] + ([out[3].clone()] if scheme != "const" else [])

    prop.set_tiling(8, 8)
    ref = gradient()
    prop.set_tiling()
    seen = []
    for tile in _tiles(prop, 10, roles):
        print(f"case: gradient {scheme} SO{so} vector tile {tile}", flush=True)
        assert _same(gradient(), ref), tile
        seen.append(tile)
    assert len(seen) >= 3


@pytest.mark.parametrize("so", range(2, 21, 2))
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_every_2d_tile_and_step_count_is_bitwise_single_steps(monkeypatch, dtype, so):
    for bc, n, nbl in ((None, (75, 130), ((3, 9), (11, 2))), (ODD[:2], (73, 131), ((0, 7), (0, 0)))):
        prop, wav = _prop(n, so, 18, nbl, "const", dtype, bc)
        with monkeypatch.context() as m:
            m.setattr(prop, "_scratch", lambda graph: None)
            ref = {k: _run(prop, wav, 2 * k) for k in range(2, 9)}
        seen = []
        for tile in range(5):
            for steps in range(2, 9):
                try:
                    prop.set_launch(tile, steps)
                except SimwaveError as e:
                    assert L.STATUS[e.status] == "SW_ERR_UNSUPPORTED"
                    continue
                assert (prop.launch()["kind"], prop.launch()["tile"], prop.launch()["steps"]) == ("steps", tile, steps)
                print(f"case: 2D {dtype} SO{so} tile {tile}, {steps} steps per launch, mirror sides {bc is not None}", flush=True)
                assert _same(_run(prop, wav, 2 * steps), ref[steps]), (tile, steps, bc)     # two launches of `steps`
                seen.append(steps)
        assert seen or so > (20 if dtype == "float32" else 14)


@pytest.mark.parametrize("n,so,scheme,dtype,bc,kind", [
    ((60, 70, 80), 2, "const", "float32", None, "vector"),
    ((9, 7, 5), 8, "const", "float32", None, "vector"),
    ((1, 40, 40), 4, "const", "float32", None, "vector"),
    ((200, 130, 257), 8, "const", "float32", None, "vector"),
    ((150, 160, 170), 6, "const", "float32", ODD, "vector"),
    ((70, 44, 58), 20, "const", "float32", ODD, "vector"),
    ((60, 71, 83), 2, "const", "float64", ODD, "vector"),
    ((38, 41, 59), 20, "const", "float64", None, "vector"),
    ((60, 70, 80), 2, "vd_staggered", "float32", None, "block"),
    ((45, 33, 61), 4, "vd_staggered", "float32", ODD, "vector"),
    ((200, 130, 257), 8, "vd_staggered", "float32", None, "vector"),
    ((60, 50, 90), 16, "vd_staggered", "float32", None, "vector"),
    ((70, 44, 58), 20, "vd_staggered", "float32", None, "block"),
    ((60, 70, 80), 2, "vd_centred", "float32", None, "vector"),
    ((60, 50, 90), 16, "vd_centred", "float32", ODD, "vector"),
    ((70, 44, 58), 20, "vd_centred", "float32", None, "vector"),
    ((97, 130), 4, "const", "float32", None, "steps"),
    ((44, 70), 20, "const", "float32", ODD[:2], "steps"),
    ((90, 47), 12, "const", "float64", None, "steps"),
    ((90, 47), 16, "const", "float64", None, "block"),
    ((97, 130), 8, "vd_staggered", "float32", None, "block"),
])
def test_kernels_that_the_library_chooses(n, so, scheme, dtype, bc, kind):
    prop, _ = _prop(n, so, 5, 4, scheme, dtype, bc)
    assert prop.launch()["kind"] == kind
    gradient = dtype == "float32" and bc is None and scheme != "vd_centred" and len(n) == 3
    for role in ("recompute", "image", "image_pair") if gradient else ():
        assert prop.launch(role)["kind"] == kind


def _choice(n, so, scheme, dtype, bc, nbl=0):
    h = (10.0,) * len(n)
    launch = Propagator(n, h, so, 0.4 * critical_dt(h, so, 3000.0), 5, scheme=scheme, nbl=nbl, dtype=dtype, bc=bc).launch()
    return (launch["kind"], launch["rows"], launch["cols"])


ALL = (("neumann", "dirichlet"), ("dirichlet", "dirichlet"), ("dirichlet", "dirichlet"))


@pytest.mark.parametrize("n,so,dtype,bc,want", [
    # us per step of the choice, of another vector tile that a model without these sides or orders took, of the scalar tiles
    ((768, 532, 507), 18, "float32", ALL, ("vector", 24, 128)),     # 958, 1373, 1041
    ((438, 574, 369), 18, "float32", ALL, ("vector", 24, 128)),     # 437, 623, 511
    ((466, 495, 397), 20, "float32", ALL, ("block", 8, 64)),        # 558, 671, 557
    ((138, 179, 137), 20, "float32", ALL, ("vector", 16, 64)),      # 45, 54, 78
    ((178, 325, 319), 2, "float64", ALL, ("vector", 12, 128)),      # 106, 131, 110
    ((207, 801, 801), 2, "float64", ALL, ("vector", 12, 128)),      # 853, 885, -
    ((713, 601, 378), 2, "float32", None, ("block", 8, 64)),        # 499, 528, 492
    ((592, 592, 592), 8, "float32", None, ("vector", 24, 128)),     # 618, -, 649
])
def test_constant_density_choices(n, so, dtype, bc, want):
    assert _choice(n, so, "const", dtype, bc) == want


@pytest.mark.parametrize("n,so,scheme,want", [
    # us per step of the choice, of the vector tile that a rule by size took, of the scalar tiles
    ((287, 272, 476), 12, "vd_staggered", ("block", 8, 64)),        # 437, 466, 436
    ((340, 340, 340), 12, "vd_staggered", ("vector", 32, 32)),      # 426, -, 502
    ((592, 592, 592), 8, "vd_staggered", ("vector", 16, 128)),      # 1287, -, 1349
    ((359, 324, 256), 14, "vd_centred", ("vector", 8, 64)),         # 214, 274, 253
    ((328, 433, 436), 6, "vd_centred", ("vector", 8, 64)),          # 287, 334, 315
    ((280, 280, 280), 8, "vd_centred", ("vector", 32, 32)),         # 122, -, 148
    ((510, 311, 457), 2, "vd_centred", ("block", 8, 64)),           # 307, 323, 307
])
def test_variable_density_choices(n, so, scheme, want):
    assert _choice(n, so, scheme, "float32", None) == want


def test_the_search_for_a_launch_runs_once_per_plan():
    # 66000 chunk counts for each tile: several ms a search
    prop = Propagator((200000, 30, 30), H, 8, 1e-4, 5, nbl=0)
    first = prop.launch()
    times = []
    for _ in range(5):
        t = time.perf_counter()
        assert prop.launch() == first
        times.append(time.perf_counter() - t)
    assert first["kind"] == "vector" and min(times) < 1e-3


@pytest.mark.parametrize("so", range(2, 21, 2))
def test_every_batch_tile_is_bitwise_the_single_shots(so):
    from paper_2201_05278_amd import Batch
    print(f"case: batch tiles SO{so}", flush=True)
    sets = [_prop(n, so, 6, 3) for n in ((25, 40, 71), (31, 22, 130))]
    ref = [p.forward(w).traces.clone() for p, w in sets]
    batch = Batch([p for p, _ in sets])
    for tile in (None, (16, 4, 9), (16, 4, 9, 0), (16, 4, 9, 1, 2), (8, 4, 7), (24, 8), (32, 8, 11, 0, 2)):
        batch.set_tiling(*tile) if tile else batch.set_tiling()
        for a, b in zip(batch.forward([w for _, w in sets]), ref):
            assert float(b.abs().max()) > 0.0 and torch.equal(a, b), tile
