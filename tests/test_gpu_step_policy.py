"""The single-step kernel's variants, bit for bit: walls in it against the tile kernel, on rows that
give a thread one node and several (16-bit storage: two or four where the row holds whole blocks)
and on a box whose steps bypass the caches."""
import pytest

from tests.gpu_util import gpu_sim

pytestmark = pytest.mark.gpu


def _state(nx, ny):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + ny)
    return (1.0 + 0.1 * (2.0 * torch.rand(9, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1.0)) / 9.0


def _run(nx, ny, model, storage, pattern, steps, f0, **kw):
    sim = gpu_sim(nx, ny, 0.4, 0.05, model, storage, pattern, **kw)
    sim.set_populations(f0)
    for _ in range(steps):
        sim.step(1)
    f = sim.populations()
    sim.close()
    return f


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(3, 2), (65, 7), (512, 5), (513, 5), (1023, 9), (1024, 33)])
def test_walls_in_single_steps_match_tiles(nx, ny, storage):
    import torch
    f0 = _state(nx, ny)
    for model in ("bgk", "uc", "partial", "complete"):
        a = _run(nx, ny, model, storage, "ab", 5, f0, walls=True)
        b = gpu_sim(nx, ny, 0.4, 0.05, model, storage, "ab", walls=True)
        b.set_populations(f0)
        b.step(5)
        assert torch.equal(a, b.populations()), model


@pytest.mark.parametrize("storage,nx,ny", [("f32", 2300, 2300), ("f16", 4096, 2560)])
def test_walls_on_boxes_beyond_the_cache(storage, nx, ny):
    """Interior as without walls: after k steps the nodes k columns away from them agree."""
    import torch
    f0 = _state(nx, ny)
    a = _run(nx, ny, "partial", storage, "ab", 3, f0, walls=True)
    b = gpu_sim(nx, ny, 0.4, 0.05, "partial", storage, "ab", walls=True)
    b.set_populations(f0)
    b.step(3)
    assert torch.equal(a, b.populations())
    free = _run(nx, ny, "partial", storage, "ab", 3, f0)
    assert torch.equal(a[:, :, 4:-4], free[:, :, 4:-4])


@pytest.mark.parametrize("storage,nx,ny", [("f32", 3072, 3000), ("f32", 3100, 3300), ("f64", 2112, 2200),
                                           ("f16", 4224, 4224), ("f16", 4500, 4520), ("bf16", 4224, 4224),
                                           ("bf16", 4700, 4400)])
def test_aa_beyond_the_cache_matches_ab(storage, nx, ny):
    """AA in place, on rows with and without padding whose buffer bypasses the caches, against A-B:
    both phases and the step after them."""
    import torch
    f0 = _state(nx, ny)
    assert torch.equal(_run(nx, ny, "complete", storage, "aa", 3, f0), _run(nx, ny, "complete", storage, "ab", 3, f0))
