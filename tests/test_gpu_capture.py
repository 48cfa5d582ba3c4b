"""Captured calls of lbm_step, replayed between the program's own eager calls and compared bit for
bit with a context that is never captured. A replay goes on from the buffer that the capture read,
so it advances the state only if the captured calls end in the buffer they started from."""
import pytest

import lbm_inputs as inp
from tests.gpu_util import gpu_sim

pytestmark = pytest.mark.gpu


def _pair(nx, ny, storage, pattern="ab", **kw):
    """Two equal contexts, the first on a stream of its own that can be captured."""
    import torch
    fields = inp.taylor_green(nx, ny, 0.05, 0.4, noise=1e-3, seed=nx)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = gpu_sim(nx, ny, 0.4, 0.02, "complete", storage, pattern, fields=fields, **kw)
    return s, a, gpu_sim(nx, ny, 0.4, 0.02, "complete", storage, pattern, fields=fields, **kw)


def _capture(s, calls):
    import torch
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        calls()
    return g


def _replay(s, g):
    import torch
    with torch.cuda.stream(s):
        g.replay()
    s.synchronize()


def _equal(s, a, b):
    import torch
    with torch.cuda.stream(s):
        f = a.populations()
    s.synchronize()
    return torch.equal(f, b.populations())


@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("stride", [8, 3])
@pytest.mark.parametrize("pattern", ["ab", "aa"])
def test_replays_past_a_recorded_run_advance(pattern, stride, adjoint):
    """The state at t = record_steps lies in a population buffer and the reverse sweep leaves it
    there, so a graph captured after the window goes on from its own result."""
    import torch
    s, a, b = _pair(200, 130, "f32", pattern, record_steps=8, ckpt_stride=stride)
    with torch.cuda.stream(s):
        a.step(8)
        if adjoint:
            w = torch.ones(9, 130, 200, device="cuda")
            first = a.adjoint_populations(w)
            assert torch.equal(first, a.adjoint_populations(w))
    b.step(8)
    g = _capture(s, lambda: (a.step(1), a.step(1)))
    for _ in range(3):
        _replay(s, g)
        b.step(2)
        assert _equal(s, a, b)


# Calls whose launches, lbm_steps_per_launch steps each, are even in number (AA: whose steps are):
# boxes on which the plans take tiles, one block for the whole box, walls, the marching kernel, and
# (512 x 2000) single steps.
CALLS = [(64, 64, "f64", {}, (16,)), (200, 130, "f32", {}, (2,)), (7, 90, "f64", {}, (64,)),
         (256, 256, "f32", {}, (20,)), (256, 256, "f32", {}, (3, 1)), (801, 3, "f64", dict(walls=True), (16,)),
         (2041, 1200, "f32", {}, (2,)), (2041, 1200, "bf16", {}, (5, 1)), (2048, 1100, "f32", {}, (4,)),
         (2048, 1100, "f64", {}, (3,)), (2048, 1100, "f32", {}, (1, 2)), (512, 2000, "f16", {}, (3,)),
         (512, 100, "f32", dict(two_step=1), (4,)), (512, 100, "f32", dict(two_step=-1), (10,)),
         (200, 130, "f32", dict(pattern="aa"), (3, 1))]


@pytest.mark.parametrize("nx,ny,storage,kw,calls", CALLS)
def test_captured_calls_replay(nx, ny, storage, kw, calls):
    """The rule of lbm_step's documentation, with the same calls made eagerly between replays."""
    s, a, b = _pair(nx, ny, storage, **kw)
    spl = a.steps_per_launch
    assert sum(calls if kw.get("pattern") == "aa" else ((n + spl - 1) // spl for n in calls)) % 2 == 0

    def run(sim):
        for n in calls:
            sim.step(n)

    g = _capture(s, lambda: run(a))
    for k in range(4):
        if k == 2:
            run(a)
        else:
            _replay(s, g)
        s.synchronize()
        run(b)
        assert _equal(s, a, b), k


def test_captured_readout_follows_eager_steps():
    """A captured readout alone: eager calls of an even count leave the state in its buffer."""
    import torch
    s, a, b = _pair(200, 130, "f32")
    out = []
    g = _capture(s, lambda: out.append(a.populations()))
    for n in (2, 8, 20):
        a.step(n)
        s.synchronize()
        _replay(s, g)
        b.step(n)
        assert torch.equal(out[0], b.populations()), n
