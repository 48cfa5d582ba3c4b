"""Several steps per launch (the tile and the marching kernels) against single-step launches
(two_step = -1), bit for bit: the collision is the same and values wait rounded to the storage
type, so any difference is an indexing error. Widths and heights at which tiles and strips end,
wrap or do not fit: 1 and 2 nodes, whole wavefronts and one more or less, odd widths around the
narrowest the marching kernel takes (124 nodes) and with strips of reduced width, boxes of one
tile and of many, and boxes large enough that the marching kernel is the planner's choice."""
import numpy as np
import pytest

import lbm_inputs as inp
from tests.gpu_util import gpu_sim

pytestmark = pytest.mark.gpu

SMALL = [(1, 1), (1, 200), (2, 3), (3, 1), (7, 90), (63, 64), (65, 33), (128, 128), (123, 70), (200, 201), (800, 1),
         (801, 3), (515, 260)]
# Boxes on which the planner takes the marching kernel (odd widths: the last strip shifted to the
# row's end, 2041 = 17 * 120 + 1 with narrower strips), and long thin ones.
LARGE = [(2048, 1100), (2041, 1200), (2047, 1031), (1999, 1301), (125, 40000), (124, 40001)]


def _state(nx, ny, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return (1.0 + 0.1 * (2.0 * torch.rand(9, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1.0)) / 9.0


def _pair(nx, ny, model, storage, **kw):
    f0 = _state(nx, ny, 100 * nx + ny)
    out = []
    for ts in (0, -1):
        sim = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", two_step=ts, **kw)
        sim.set_populations(f0)
        out.append(sim)
    return out


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", SMALL)
def test_small_boxes_match_single_steps(nx, ny, storage):
    import torch
    for model in ("bgk", "uc", "partial", "complete"):
        a, b = _pair(nx, ny, model, storage)
        for n in (2, 3, 5, 8, 17):
            a.step(n)
            b.step(n)
            assert torch.equal(a.populations(), b.populations()), (model, n, a.time)
        assert all(torch.equal(u, v) for u, v in zip(a.moments(), b.moments()))


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", LARGE)
def test_large_boxes_match_single_steps(nx, ny, storage):
    import torch
    a, b = _pair(nx, ny, "bgk" if storage == "f16" else "complete", storage)
    for n in (4, 5, 6, 7):
        a.step(n)
        b.step(n)
        assert torch.equal(a.populations(), b.populations()), n


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny", [(3, 1), (3, 5), (31, 64), (800, 1), (300, 200)])
def test_walls_match_single_steps(nx, ny, storage):
    import torch
    for model in ("bgk", "partial"):
        a, b = _pair(nx, ny, model, storage, walls=True)
        for n in (2, 3, 11, 40):
            a.step(n)
            b.step(n)
            assert torch.equal(a.populations(), b.populations()), (model, n)


@pytest.mark.parametrize("storage", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("nx,ny", [(1, 9), (33, 20), (125, 70), (300, 257), (1401, 1100), (1408, 900)])
def test_recorded_sweep_matches_single_steps(nx, ny, storage):
    """Forward states, the moment records (through the adjoint) and the reverse sweep: N = 11 in
    segments of 11 (one launch more than any plan's steps), 4 and 1. The collision's VJP writes
    out its fused products, so the sweeps agree bit for bit too."""
    import torch
    f0 = _state(nx, ny, 5)
    w = torch.as_tensor(inp.random_direction((9, ny, nx), seed=6), device="cuda")
    for model in ("bgk", "uc", "partial", "complete") if nx < 200 else ("complete",):
        for stride in (11, 4, 1):
            got = []
            for ts in (0, -1):
                sim = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", two_step=ts, record_steps=11, ckpt_stride=stride)
                sim.set_populations(f0)
                sim.step(11)
                got.append((sim.populations(), sim.adjoint_populations(w), sim.adjoint_populations(w), sim.populations()))
                sim.step(3)  # past the window, from the state the sweep gave back
                got[-1] += (sim.populations(),)
                sim.close()
            for k, (u, v) in enumerate(zip(*got)):
                assert torch.equal(u, v), (model, stride, k)
            assert torch.equal(got[0][1], got[0][2]) and torch.equal(got[0][0], got[0][3])


def test_steps_in_a_captured_graph():
    """lbm_step only launches kernels: a captured graph of it replays like eager calls (an even
    number of launches, so the buffers are back in their places)."""
    import torch
    nx, ny = 130, 77
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a, b = _pair(nx, ny, "complete", "f32")
        a.step(16)
        g = torch.cuda.CUDAGraph()
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            a.step(16)
            a.step(16)
        b.step(16)
        for _ in range(3):
            g.replay()
            s.synchronize()
            b.step(32)
            assert torch.equal(a.populations(), b.populations())
    assert np.isfinite(a.populations().sum().item())
