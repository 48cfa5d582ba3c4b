"""Which kernel a context launches (lbm_next_launch, MI355X), and bit-for-bit comparisons on boxes
where that kernel is known to run: sizes from the launch plans, asserted, so that a change of the
plans cannot leave a comparison of single steps with themselves."""
import numpy as np
import pytest

import lbm_inputs as inp
import oracle
from tests.gpu_util import gpu_sim
from tests.lbm_diag import eps_f

pytestmark = pytest.mark.gpu

STEP, MARCH, TILE, PAIR = 0, 1, 2, 3


def _next(sim, n, reverse=False):
    from paper_2602_21242_amd import capi
    s, kernel, steps = capi.lbm_next_launch(sim._ctx, n, reverse)
    capi.check(s, "lbm_next_launch")
    return kernel, steps


def _state(nx, ny):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(3 * nx + ny)
    return (1.0 + 0.1 * (2.0 * torch.rand(9, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1.0)) / 9.0


def test_kernels_of_known_boxes():
    cases = [((48, 20, "f64", {}), 64, TILE, None), ((1, 200, "f64", {}), 4000, TILE, 4000), ((48, 20, "f64", dict(two_step=-1)), 64, STEP, 1),
             ((48, 20, "f32", dict(pattern="aa")), 64, STEP, 1), ((1024, 1024, "f32", {}), 100, TILE, 5),
             ((1024, 1024, "f32", {}), 2, PAIR, 2), ((4096, 4096, "f32", {}), 100, MARCH, 4), ((4096, 4096, "f32", {}), 2, PAIR, 2),
             ((4096, 4096, "f32", {}), 1, STEP, 1), ((2048, 2048, "f64", {}), 2, PAIR, 2), ((4096, 4096, "f16", {}), 2, MARCH, 2),
             ((8192, 8192, "f16", {}), 100, MARCH, 3), ((1024, 1024, "f16", {}), 2, STEP, 1), ((800, 1, "f64", dict(walls=True)), 50, TILE, None),
             ((512, 100, "f32", dict(two_step=1)), 100, PAIR, 2)]
    for (nx, ny, storage, kw), n, kernel, steps in cases:
        sim = gpu_sim(nx, ny, 0.4, 0.02, "complete", storage, **kw)
        got = _next(sim, n)
        assert got[0] == kernel and steps in (None, got[1]) and 1 <= got[1] <= n, (nx, ny, storage, kw, n, got)
        sim.close()
    sim = gpu_sim(64, 64, 0.4, 0.02, "complete", "f32", record_steps=8)
    assert _next(sim, 3, reverse=True)[0] == TILE
    from paper_2602_21242_amd import capi
    assert capi.lbm_next_launch(sim._ctx, 0)[0] == capi.LBM_ERR_INVALID_ARGUMENT
    assert capi.lbm_next_launch(gpu_sim(64, 64, 0.4, 0.02, "complete", "f32")._ctx, 1, True)[0] == capi.LBM_ERR_STATE


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(2041, 1600), (3251, 2191), (2521, 1999), (125, 90000)])
def test_odd_widths_march(nx, ny, storage):
    """Two nodes per lane on odd widths: the last strip shifted to the row's end, narrower strips,
    and two strips that overlap almost entirely (125 nodes; tiles or marches by storage type)."""
    import torch
    model = "complete"
    f0 = _state(nx, ny)
    a = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", f0=f0)
    b = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", f0=f0, two_step=-1)
    if nx != 125:
        assert _next(a, 100)[0] == MARCH
    for n in (4, 5, 6):
        a.step(n)
        b.step(n)
        assert torch.equal(a.populations(dtype=torch.float32), b.populations(dtype=torch.float32)), n


@pytest.mark.parametrize("storage", ["f16", "bf16", "f32", "f64"])
@pytest.mark.parametrize("nx,ny,stride,reverse", [(512, 512, 6, TILE), (512, 512, 11, TILE), (1501, 1300, 11, MARCH),
                                                  (1536, 1100, 4, TILE)])
def test_recorded_launches(nx, ny, stride, reverse, storage):
    """Records of forward launches and reverse launches of both kinds, 16-bit storage among them,
    against single steps; 512 x 512 in segments of six takes FP32 reverse tiles of two nodes per
    thread."""
    import torch
    f0 = _state(nx, ny)
    w = torch.as_tensor(inp.random_direction((9, ny, nx), seed=6), device="cuda")
    got = []
    for ts in (0, -1):
        sim = gpu_sim(nx, ny, 0.4, 0.05, "complete", storage, "ab", two_step=ts, record_steps=11, ckpt_stride=stride)
        if ts == 0 and storage != "f64":
            assert _next(sim, stride, reverse=True)[0] == reverse
        sim.set_populations(f0)
        sim.step(11)
        got.append((sim.populations(), sim.adjoint_populations(w)))
        sim.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_ab_graph_replays_match_single_launches(storage):
    """A-B contexts of one step per launch on launch-bound grids replay a recorded graph of 64 steps,
    from either buffer, between single steps, readouts and synchronisations: bit for bit against a
    context advanced one lbm_step(1) call at a time (never a graph), then with the oracle."""
    import torch
    nx, ny, th, nu = 48, 20, 0.4, 0.02
    fields = inp.taylor_green(nx, ny, 0.05, th, noise=1e-3, seed=4)
    a = gpu_sim(nx, ny, th, nu, "complete", storage, "ab", fields=fields, two_step=-1)
    b = gpu_sim(nx, ny, th, nu, "complete", storage, "ab", fields=fields, two_step=-1)
    assert _next(a, 64) == (STEP, 1)
    total = 0
    for chunk, extra in ((64, 1), (128, 0), (64, 3), (192, 1)):
        a.step(chunk)
        a.moments()
        torch.cuda.synchronize()
        for _ in range(chunk):
            b.step(1)
        total += chunk
        assert a.time == b.time == total
        assert torch.equal(a.populations(), b.populations()), (chunk, total)
        a.step(extra)
        b.step(extra)
        total += extra
    ref = oracle.run(oracle.init_equilibrium(*fields, th), th, nu, "complete", total)
    assert eps_f(a.populations().cpu().numpy(), ref) <= {"f64": 1e-12, "f32": 1e-5, "f16": 1e-3}[storage]
    assert np.isfinite(ref).all()
