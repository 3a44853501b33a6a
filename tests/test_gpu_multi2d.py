"""2D forward runs in launches of several steps, bitwise against the single-step kernels (which the oracle tests pin)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FREE = (("neumann", "dirichlet"), ("dirichlet", "neumann"))


def _run(monkeypatch, multi, n, so, nbl, steps, dtype, bc, src, interp, stride, every=0, graph=False, offset=0, step0=0):
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    h = (10.0, 12.5)
    rng = np.random.default_rng(so + n[0])
    vel = torch.from_numpy(rng.uniform(1500.0, 3000.0, n)).float().to(torch.float64 if dtype == "float64" else torch.float32)
    dt = 0.7 * critical_dt(h, so, 3000.0)
    prop = Propagator(n, h, so, dt, steps + step0, nbl=nbl, bc=bc, dtype=dtype)
    prop.set_sources(np.asarray(src) * np.asarray(h), interp)
    prop.set_receivers([[h[0] * z, h[1] * y] for z, y in ((6.0, 7.3), (n[0] - 8.4, n[1] - 7.0), (n[0] / 2, n[1] / 2))], interp)
    prop.prepare(vel, cmax=3000.0)
    wav = torch.stack([ricker(25.0 + 3.0 * k, dt, steps + step0) for k in range(len(src))], 1)
    if not multi:
        monkeypatch.setattr(prop, "_scratch", lambda use_graph: None)
    size = prop.layout.field_elems
    store = [torch.zeros(size + 4, dtype=prop.torch_dtype, device="cuda") for _ in range(2)]
    fields = tuple(s[offset:offset + size] for s in store)
    if step0:                                   # resume from a wavefield that is not at rest
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        for f in fields:
            v = prop.grid_view(f)
            v.copy_(torch.randn(tuple(v.shape), generator=g, device="cuda", dtype=v.dtype))
    kw = {} if dtype == "float64" else {"checkpoint_every": every, "use_graph": graph}
    for _ in range(3 if graph else 1):          # replays with eager work between them
        res = prop.forward(wav, saving_stride=stride, fields=fields, step0=step0, **kw)
        torch.cuda.synchronize()
        kw.setdefault("traces", res.traces)
    cur = res.current
    out = [res.traces, prop.grid_view(res.fields[cur]), prop.grid_view(res.fields[1 - cur])]
    out += [t for t in (res.snaps, res.ckpt) if t is not None]
    return [t.clone() for t in out], prop


@pytest.mark.parametrize("n,so,nbl,steps,dtype,bc,interp,stride,every,graph", [
    ((31, 33), 2, 0, 17, "float32", None, "linear", 3, 0, False),           # one tile, no layer, odd extents
    ((97, 130), 4, 7, 33, "float32", None, "hicks", 0, 5, False),           # checkpoints inside launches
    ((97, 130), 4, 7, 33, "float32", FREE, "hicks", 0, 5, False),           # checkpoints with mirror sides: single steps
    ((97, 131), 4, 7, 33, "float32", FREE, "hicks", 0, 0, False),
    ((160, 301), 8, 12, 24, "float32", FREE, "hicks", 5, 0, True),          # graph, several tiles, snapshots
    ((420, 1000), 8, 20, 9, "float32", None, "hicks", 0, 4, False),         # a step before the launches
    ((64, 64), 12, 9, 7, "float32", FREE, "linear", 0, 0, False),
    ((75, 91), 16, 8, 13, "float32", None, "hicks", 2, 6, False),
    ((44, 70), 20, 10, 10, "float32", FREE, "hicks", 0, 0, False),          # two steps per launch
    ((33, 57), 2, 5, 19, "float64", FREE, "linear", 4, 0, False),
    ((140, 333), 8, 11, 22, "float64", None, "hicks", 0, 0, False),
    ((90, 47), 12, 13, 8, "float64", FREE, "hicks", 3, 0, False),
    ((50, 50), 8, 6, 4, "float32", None, "hicks", 0, 0, False),             # the fewest steps
    ((50, 50), 8, 6, 3, "float32", None, "hicks", 0, 0, False),             # too few: single steps
])
def test_several_steps_per_launch_are_bitwise_single_steps(monkeypatch, n, so, nbl, steps, dtype, bc, interp, stride, every,
                                                           graph):
    print(f"case: 2D {n} SO{so} {dtype} {bc} {interp} steps {steps}", flush=True)
    src = [(9.3, n[1] / 2 + 0.4), (9.8, n[1] / 2 + 2.0), (n[0] / 2, 8.5)]
    args = (n, so, nbl, steps, dtype, bc, src, interp, stride, every, graph)
    a, prop = _run(monkeypatch, True, *args)
    assert prop._scratch(False) is not None
    b, _ = _run(monkeypatch, False, *args)
    assert len(a) == len(b) and float(a[1].abs().max()) > 0.0
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_resume_and_buffers_off_16_bytes(monkeypatch):
    print("case: 2D resume at a step, and fields aligned to 4 bytes only", flush=True)
    args = ((120, 150), 8, 9, 21, "float32", FREE, [(9.3, 70.4)], "hicks", 0)
    a, _ = _run(monkeypatch, True, *args, step0=6)
    b, _ = _run(monkeypatch, False, *args, step0=6)
    c, _ = _run(monkeypatch, True, *args, step0=6, offset=1)      # left to the single-step kernels
    for x, y, z in zip(a, b, c):
        assert torch.equal(x, y) and torch.equal(x, z)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_runs_without_receivers_keep_only_the_levels_that_are_read(monkeypatch, dtype):
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    n, h, so, steps = (120, 170), (10.0, 12.5), 4, 29
    dt = 0.7 * critical_dt(h, so, 3000.0)
    wav = ricker(25.0, dt, steps).reshape(-1, 1)
    for kw in ({}, {"saving_stride": 3}) + (({"checkpoint_every": 5}, {"saving_stride": 4, "checkpoint_every": 7})
                                            if dtype == "float32" else ()):
        print(f"case: 2D without receivers {dtype} {kw}", flush=True)
        out = []
        for multi in (True, False):
            prop = Propagator(n, h, so, dt, steps, nbl=9, dtype=dtype)
            prop.set_sources([[605.0, 1061.0]], "hicks")
            prop.prepare(torch.full(n, 2500.0, dtype=prop.torch_dtype), cmax=3000.0)
            if not multi:
                monkeypatch.setattr(prop, "_scratch", lambda run: None)
            assert prop.launch()["steps"] > 2
            r = prop.forward(wav, **kw)
            out.append([prop.grid_view(f) for f in r.fields] + [t for t in (r.snaps, r.ckpt) if t is not None])
        assert float(out[0][0].abs().max()) > 0.0
        for a, b in zip(*out):
            assert torch.equal(a, b)
