"""Which device scratch the binding hands to 2D forwards (no GPU: the library's launch is replaced by a recorder)."""
import pytest
import torch

from paper_2201_05278_amd import Propagator
from paper_2201_05278_amd import _lib as L
from paper_2201_05278_amd import propagator as P


class _Recorder:
    """The library, with the forward entry points recording their scratch."""

    def __init__(self, real):
        self.real, self.calls = real, []

    def __getattr__(self, name):
        if name not in ("sw_forward_scratch", "sw_forward_f64_scratch"):
            return getattr(self.real, name)

        def call(plan, io, scratch, nbytes, stream):
            self.calls.append((scratch.value, nbytes))
            return 0
        return call


@pytest.fixture
def recorder(monkeypatch):
    rec = _Recorder(L.lib())
    monkeypatch.setattr(L, "lib", lambda: rec)
    monkeypatch.setattr(P, "_stream", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: None)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda self, stream: None)
    return rec


def _prop(n=(60, 80), so=8, receivers=True, dtype="float32", **kw):
    prop = Propagator(n, (10.0, 10.0), so, 1e-4, 20, nbl=8, device="cpu", dtype=dtype, **kw)
    prop.set_sources([[300.0, 400.0]], "linear")
    if receivers:
        prop.set_receivers([[100.0, 100.0]], "linear")
    prop._vel = torch.zeros(n)                   # (prepare() needs a device)
    return prop


def test_graphs_over_other_wavefields_have_a_scratch_of_their_own(recorder):
    prop, wav = _prop(), torch.zeros(20, 1)
    pairs = [(prop.new_field(), prop.new_field()) for _ in range(2)]
    held = []                                    # as while both graphs are in flight: nothing is handed out twice
    for fields in (pairs[0], pairs[0], pairs[1]):
        prop.forward(wav, use_graph=True, fields=fields)
        held.append(prop._graph_scratch)
    (a, na), (b, nb), (c, nc) = recorder.calls
    assert a and na == nb == nc > 0
    assert a == b                                # a replay finds the scratch its graph was captured with
    assert c != a


@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_a_run_asks_for_the_levels_it_needs_and_gives_them_back(recorder, dtype):
    wav, sizes = torch.zeros(20, 1), {}
    for receivers in (True, False):
        prop = _prop(receivers=receivers, dtype=dtype)
        steps, field = prop.launch()["steps"], prop.layout.field_elems * (4 if dtype == "float32" else 8)
        assert steps > 2
        for stride in (0, 5):
            recorder.calls.clear()
            prop.forward(wav, saving_stride=stride)
            sizes[receivers, stride] = recorder.calls[0][1] // field
            assert recorder.calls[0][0]
            kept = [t for t in prop.__dict__.values() if isinstance(t, torch.Tensor)]
            for item in prop._keep:
                kept += item if isinstance(item, tuple) else [item]
            assert not any(t is not None and t.dtype == torch.uint8 for t in kept)      # nothing holds the scratch
    full = 2 + 2 * (steps - 2)
    assert sizes == {(True, 0): full, (True, 5): full, (False, 5): full, (False, 0): 2}


def test_a_run_too_short_for_a_launch_asks_for_nothing(recorder):
    prop, wav = _prop(), torch.zeros(20, 1)
    for steps in (1, 3, 4):
        prop.forward(wav, step0=2, nsteps_run=steps)
    assert [bool(p) for p, _ in recorder.calls] == [False, False, True]
    assert recorder.calls[0][1] == 0


@pytest.mark.parametrize("side,wants", [("none", True), ("neumann", False), ("dirichlet", False)])
def test_checkpoints_that_need_single_steps_ask_for_nothing(recorder, side, wants):
    prop, wav = _prop(bc=[(side, "none"), ("none", "none")]), torch.zeros(20, 1)
    prop.forward(wav, checkpoint_every=5)
    prop.forward(wav, saving_stride=5)
    assert [bool(p) for p, _ in recorder.calls] == [wants, True]
