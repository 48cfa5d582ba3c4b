"""Calls of two steps, whose launches have a plan of their own (the pair kernel beyond the cache,
marches in strips with a narrow halo, wide tiles, single steps), bit for bit against single steps:
boxes on which each is taken, odd widths and short columns among them."""
import pytest

from tests.gpu_util import gpu_sim

pytestmark = pytest.mark.gpu

BOXES = [(128, 128), (384, 384), (512, 512), (513, 200), (1000, 600), (1024, 1024), (125, 9000), (127, 9001),
         (1447, 901), (2041, 1200), (1024, 4500), (4608, 1200), (2560, 2049), (512, 20000), (16384, 333)]


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", BOXES)
def test_calls_of_two_steps(nx, ny, storage):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + ny)
    f0 = (1.0 + 0.1 * (2.0 * torch.rand(9, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1.0)) / 9.0
    for model in ("complete",) if nx * ny > 1 << 20 else ("bgk", "complete"):
        a = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", f0=f0)
        b = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", f0=f0, two_step=-1)
        for n in (2, 2, 6, 7):
            a.step(n)
            b.step(n)
            assert torch.equal(a.populations(), b.populations()), (model, n)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny", [(2048, 2200), (6144, 768), (1024 * 1024, 5), (1024 * 2048, 2), (1024 * 4096, 1)])
@pytest.mark.parametrize("model", ["bgk", "uc", "partial", "complete"])
def test_pair_kernel(nx, ny, storage, model):
    """Row blocks of several heights, blocks that wrap in x, columns of one, two and five rows."""
    import torch
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, :]
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[:, None]
    fields = (1.0 + 0.01 * torch.cos(0.7 * x + 0.3 * y), 0.05 * torch.sin(0.9 * x - 1.1 * y), 0.04 * torch.cos(1.3 * x + 2.1 * y))
    out = []
    for ts in (0, -1):
        sim = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", fields=fields, two_step=ts)
        if ts == 0:
            assert sim.steps_per_launch == 2
        sim.step(2)
        sim.step(2)
        out.append(sim.populations(dtype=torch.float32 if storage == "f32" else torch.float64))
        sim.close()
    assert torch.equal(*out)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(384, 384), (513, 200), (700, 700), (1000, 600), (2041, 1200), (1024, 1500)])
def test_recorded_segments_of_two_steps(nx, ny, storage):
    """Forward and recomputed launches that end at checkpoints two steps apart, with records."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + ny)
    f0 = (1.0 + 0.1 * (2.0 * torch.rand(9, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1.0)) / 9.0
    w = torch.randn(9, ny, nx, generator=g, device="cuda", dtype=torch.float64)
    got = []
    for ts in (0, -1):
        sim = gpu_sim(nx, ny, 0.4, 0.05, "complete", storage, "ab", two_step=ts, record_steps=7, ckpt_stride=2)
        sim.set_populations(f0)
        sim.step(7)
        got.append((sim.populations(), sim.adjoint_populations(w)))
        sim.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
