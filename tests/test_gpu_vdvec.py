"""Vector tiles of the 3D variable-density stencils (the default tiling), bitwise against the scalar tiles (which the oracle
tests and an explicit tiling pin)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FREE = (("neumann", "dirichlet"), ("dirichlet", "neumann"), ("neumann", "none"))
ODD = (("none", "neumann"), ("none", "dirichlet"), ("dirichlet", "neumann"))


def _prop(scheme, n, so, nbl, steps, bc=None):
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    h = (10.0, 12.0, 9.0)
    dt = 0.5 * critical_dt(h, so, 3000.0)
    prop = Propagator(n, h, so, dt, steps, scheme=scheme, nbl=nbl, bc=bc)
    mid = [hh * (k - 1) / 2 for k, hh in zip(n, h)]
    prop.set_sources([mid], "linear")
    prop.set_receivers([mid, [0.9 * m for m in mid]], "linear")
    rng = np.random.default_rng(0)
    vel = torch.from_numpy(rng.uniform(1500.0, 3000.0, n)).float()
    rho = torch.from_numpy(rng.uniform(1000.0, 2500.0, n)).float()
    prop.prepare(vel, rho, cmax=3000.0)
    return prop, ricker(30.0, dt, steps).reshape(-1, 1)


@pytest.mark.parametrize("scheme", ["vd_staggered", "vd_centred"])
@pytest.mark.parametrize("n,so,nbl,bc", [
    ((60, 70, 80), 2, 5, None),
    ((45, 33, 61), 4, ((3, 9), (0, 7), (11, 2)), ODD),          # ends inside a vector, uneven layer
    ((150, 160, 170), 6, 20, FREE),
    ((200, 130, 257), 8, 8, None),
    ((33, 47, 130), 8, 0, FREE),                                # no layer
    ((9, 7, 5), 8, 4, None),                                    # smaller than a tile and than its halo
    ((1, 40, 40), 4, 0, None),                                  # a single plane
    ((80, 90, 66), 10, 7, ODD),
    ((64, 64, 63), 12, 10, None),
    ((50, 60, 129), 14, 9, FREE),
    ((60, 50, 90), 16, 12, None),
    ((40, 50, 71), 18, 6, ODD),
    ((70, 44, 58), 20, 10, FREE),
])
def test_default_tiles_are_bitwise_scalar_tiles(scheme, n, so, nbl, bc):
    print(f"case: vector tiles {scheme} {n} SO{so} {bc}", flush=True)
    steps, out = 7, []
    prop, wav = _prop(scheme, n, so, nbl, steps, bc)
    for tile in (None, (8, 8)):
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
        out.append([res.traces, fields[0], fields[1]])
    assert float(prop.grid_view(out[0][1]).abs().max()) > 0.0
    for x, y in zip(*out):                                      # whole buffers: what lies off the grid as well
        assert torch.equal(x, y)


@pytest.mark.parametrize("n,so,every", [((60, 70, 83), 4, 5), ((90, 64, 101), 8, 4), ((50, 41, 66), 16, 7), ((40, 44, 47), 20, 3)])
def test_gradients_on_default_tiles_are_bitwise_scalar_tiles(n, so, every):
    print(f"case: staggered gradient on vector tiles {n} SO{so}", flush=True)
    steps, out = 13, []
    for tile in (None, (8, 8)):
        prop, wav = _prop("vd_staggered", n, so, 9, steps)
        prop.set_tiling(*tile) if tile else prop.set_tiling()
        fw = prop.forward(wav, checkpoint_every=every)
        grad_vel, _, _, grad_rho = prop.adjoint(wav, fw.traces, fw.ckpt, every)
        out.append([grad_vel.clone(), grad_rho.clone()])
    for x, y in zip(*out):
        assert float(x.abs().max()) > 0.0
        assert torch.equal(x, y)
