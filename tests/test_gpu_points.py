"""Injection and recording in one launch: a run whose levels are recorded one step later, bitwise against the same run
called one step at a time (each call records its own level)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _prop(n, scheme, dtype, interp, nsrc, nrec, steps):
    from paper_2201_05278_amd import Propagator, critical_dt, ricker
    h = (10.0,) * len(n)
    dt = 0.5 * critical_dt(h, 4, 3000.0)
    prop = Propagator(n, h, 4, dt, steps, scheme=scheme, nbl=6, dtype=dtype)
    mid = [5.0 * (k - 1) for k in n]
    g = torch.Generator()
    g.manual_seed(5)
    span = torch.tensor([10.0 * (k - 1) for k in n])
    rec = torch.rand((max(nrec - 1, 0), len(n)), generator=g) * span
    if nsrc:
        prop.set_sources([[m + 3.0 * i for m in mid] for i in range(nsrc)], interp)
    if nrec:
        prop.set_receivers([mid] + rec.tolist(), interp)     # the first one at a source: reads what was just injected
    vel = torch.full(n, 2000.0, dtype=prop.torch_dtype)
    rho = None if scheme == "const" else torch.full(n, 1500.0)
    prop.prepare(vel, rho, cmax=3000.0) if rho is not None else prop.prepare(vel, cmax=3000.0)
    return prop, torch.stack([ricker(25.0, dt, steps)] * max(nsrc, 1), 1)


@pytest.mark.parametrize("n,scheme,dtype,interp,nsrc,nrec", [
    ((30, 33, 41), "const", "float32", "hicks", 1, 300),
    ((30, 33, 41), "const", "float64", "hicks", 3, 17),
    ((30, 33, 41), "vd_staggered", "float32", "linear", 40, 1),
    ((30, 33, 41), "vd_centred", "float32", "linear", 1, 1000),
    ((51, 61), "vd_staggered", "float32", "hicks", 2, 65),
    ((30, 33, 41), "const", "float32", "linear", 2, 0),
    ((30, 33, 41), "const", "float64", "linear", 0, 5),
])
@pytest.mark.parametrize("steps", [1, 2, 7])
def test_late_recording_is_bitwise_immediate_recording(n, scheme, dtype, interp, nsrc, nrec, steps):
    print(f"case: points {n} {scheme} {dtype} {interp} {nsrc} sources {nrec} receivers {steps} steps", flush=True)
    prop, wav = _prop(n, scheme, dtype, interp, nsrc, nrec, steps)
    f = [(prop.new_field(), prop.new_field()) for _ in range(2)]
    whole = prop.forward(wav if nsrc else None, fields=f[0]).traces
    rows = []
    for k in range(steps):
        r = prop.forward(wav if nsrc else None, fields=f[1] if k % 2 == 0 else f[1][::-1], step0=k, nsteps_run=1)
        rows.append(r.traces[k].clone() if nrec else None)
    assert torch.equal(f[0][0], f[1][0]) and torch.equal(f[0][1], f[1][1])
    if nrec:
        assert torch.equal(whole, torch.stack(rows))
        if nsrc:
            assert float(whole.abs().max()) > 0.0


@pytest.mark.parametrize("graph", [False, True])
def test_batch_records_what_single_shots_record(graph):
    from paper_2201_05278_amd import Batch
    print(f"case: points of a batch, graph {graph}", flush=True)
    steps, shots = 6, [((30, 33, 41), 1, 40), ((25, 28, 50), 3, 1), ((33, 20, 31), 0, 9), ((31, 22, 27), 2, 0)]
    made = [_prop(n, "const", "float32", "hicks", ns, nr, steps) for n, ns, nr in shots]
    alone = []
    for (prop, wav), (_, ns, nr) in zip(made, shots):
        prop.set_tiling(8, 8)
        alone.append(prop.forward(wav if ns else None).traces.clone() if nr else None)
        prop.set_tiling()
    batch = Batch([p for p, _ in made])
    for _ in range(3 if graph else 1):
        got = batch.forward([w for _, w in made], use_graph=graph)
        torch.cuda.synchronize()
        for a, b in zip(alone, got):
            if a is not None:
                assert torch.equal(a, b)
