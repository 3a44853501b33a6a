"""Vector tiles of the 3D constant-density stencil (the default tiling), bitwise against the scalar tiles (which the oracle
tests and an explicit tiling pin)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FREE = (("neumann", "dirichlet"), ("dirichlet", "neumann"), ("neumann", "none"))
ODD = (("none", "neumann"), ("none", "dirichlet"), ("dirichlet", "neumann"))


def _prop(n, so, nbl, steps, dtype="float32", bc=None, seed=0):
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    h = (10.0, 12.0, 9.0)
    dt = 0.8 * critical_dt(h, so, 3000.0)
    prop = Propagator(n, h, so, dt, steps, nbl=nbl, bc=bc, dtype=dtype)
    mid = [hh * (k - 1) / 2 for k, hh in zip(n, h)]
    prop.set_sources([mid], "linear")
    prop.set_receivers([mid, [0.9 * m for m in mid]], "linear")
    vel = torch.from_numpy(np.random.default_rng(seed).uniform(1500.0, 3000.0, n)).to(prop.torch_dtype)
    prop.prepare(vel, cmax=3000.0)
    return prop, ricker(30.0, dt, steps).reshape(-1, 1), vel


def _levels(prop, steps, wav, tile=None):
    """Traces and both levels of a run that resumes from noise on the whole grid."""
    prop.set_tiling(*tile) if tile else prop.set_tiling()
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    fields = []
    for _ in range(2):
        f = prop.new_field()
        v = prop.grid_view(f)
        v.copy_(torch.randn(tuple(v.shape), generator=g, device="cuda", dtype=v.dtype))
        fields.append(f)
    res = prop.forward(wav, fields=tuple(fields), step0=1, nsteps_run=steps - 1)
    return [res.traces, prop.grid_view(fields[0]), prop.grid_view(fields[1])]


@pytest.mark.parametrize("n,so,nbl,dtype,bc", [
    ((60, 70, 80), 2, 5, "float32", None),
    ((45, 33, 61), 4, ((3, 9), (0, 7), (11, 2)), "float32", ODD),          # ends inside a vector, uneven layer
    ((150, 160, 170), 6, 20, "float32", FREE),
    ((200, 130, 257), 8, 8, "float32", None),
    ((33, 47, 130), 8, 0, "float32", FREE),                                # no layer
    ((9, 7, 5), 8, 4, "float32", None),                                    # smaller than a tile and than its halo
    ((1, 40, 40), 4, 0, "float32", None),                                  # a single plane
    ((80, 90, 66), 10, 7, "float32", ODD),
    ((64, 64, 63), 12, 10, "float32", None),
    ((100, 60, 129), 14, 9, "float32", FREE),
    ((120, 110, 90), 16, 12, "float32", None),
    ((40, 50, 71), 18, 6, "float32", ODD),
    ((70, 44, 58), 20, 10, "float32", FREE),
    ((60, 71, 83), 2, 5, "float64", ODD),
    ((120, 130, 141), 8, 12, "float64", FREE),
    ((50, 64, 65), 10, 9, "float64", None),
    ((44, 66, 47), 16, 10, "float64", ODD),
    ((38, 41, 59), 20, 12, "float64", None),
])
def test_default_tiles_are_bitwise_scalar_tiles(n, so, nbl, dtype, bc):
    print(f"case: vector tiles {n} SO{so} {dtype} {bc}", flush=True)
    steps = 7
    prop, wav, _ = _prop(n, so, nbl, steps, dtype, bc)
    a = _levels(prop, steps, wav)
    b = _levels(prop, steps, wav, (8, 8))
    assert float(a[1].abs().max()) > 0.0
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n,so,every", [((60, 70, 83), 4, 5), ((90, 64, 101), 8, 4), ((50, 41, 66), 16, 7), ((40, 44, 47), 20, 3)])
def test_gradients_on_default_tiles_are_bitwise_scalar_tiles(n, so, every):
    print(f"case: gradient on vector tiles {n} SO{so}", flush=True)
    steps, out = 13, []
    for tile in (None, (8, 8)):
        prop, wav, _ = _prop(n, so, 9, steps)
        prop.set_tiling(*tile) if tile else prop.set_tiling()
        fw = prop.forward(wav, checkpoint_every=every)
        out.append(prop.adjoint(wav, fw.traces, fw.ckpt, every)[0].clone())
    assert float(out[0].abs().max()) > 0.0
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("so", [2, 8, 14, 20])
def test_batch_on_vector_tiles_is_bitwise_scalar_tiles(so):
    from paper_2201_05278_amd import Batch
    print(f"case: batch on vector tiles SO{so}", flush=True)
    sets = [_prop(n, so, 8, 9, seed=k) for k, n in enumerate([(50, 61, 70), (33, 90, 41), (64, 40, 129)])]
    wavs, out = [s[1] for s in sets], []
    batch = Batch([s[0] for s in sets])
    for tile in (None, (16, 4, 11), (8, 4, 13), (16, 4, 0, 1, 1, 3)):
        batch.set_tiling(*tile) if tile else batch.set_tiling()
        tr = batch.forward(wavs, use_graph=False)
        out.append([t.clone() for t in tr] + [p.grid_view(f[batch.current]).clone() for (p, _, _), f in zip(sets, batch.fields)])
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert torch.equal(x, y)


@pytest.mark.parametrize("scheme,dtype", [("const", "float32"), ("const", "float64"), ("vd_staggered", "float32"),
                                          ("vd_centred", "float32")])
def test_wavefields_at_any_element_of_a_buffer(scheme, dtype):
    """Buffers that start between 16-byte boundaries: same levels, traces and checkpoints."""
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    print(f"case: wavefields off the vector alignment {scheme} {dtype}", flush=True)
    n, h, steps, out = (40, 37, 70), (10.0, 10.0, 10.0), 9, []
    dt = 0.5 * critical_dt(h, 8, 3000.0)
    prop = Propagator(n, h, 8, dt, steps, scheme=scheme, nbl=6, dtype=dtype)
    prop.set_sources([[195.0, 180.0, 345.0]], "linear")
    prop.set_receivers([[195.0, 180.0, 345.0], [100.0, 90.0, 300.0]], "linear")
    rng = np.random.default_rng(2)
    vel = torch.from_numpy(rng.uniform(1500.0, 3000.0, n)).to(prop.torch_dtype)
    rho = torch.from_numpy(rng.uniform(1000.0, 2000.0, n)).float()
    prop.prepare(vel, *(() if scheme == "const" else (rho,)), cmax=3000.0)
    size = prop.layout.field_elems
    every = 4 if dtype == "float32" and scheme != "vd_centred" else 0
    for off in (0, 1, 3):
        f = [torch.zeros(size + 4, dtype=prop.torch_dtype, device="cuda")[off:off + size] for _ in range(2)]
        r = prop.forward(ricker(30.0, dt, steps).reshape(-1, 1), fields=tuple(f), checkpoint_every=every)
        out.append([r.traces.clone(), *f] + ([r.ckpt] if every else []))
    assert float(out[0][0].abs().max()) > 0.0
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b)
