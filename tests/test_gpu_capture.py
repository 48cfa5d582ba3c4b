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
