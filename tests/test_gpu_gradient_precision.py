"""Rounding of FP32 gradients over many steps, against the FP64 gradient of the same run."""
import math

import pytest

pytestmark = pytest.mark.gpu


def _fields(flow, nx, ny):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.arange(nx, device="cuda", dtype=torch.float64)[None, :] / nx
    y = torch.arange(ny, device="cuda", dtype=torch.float64)[:, None] / ny
    noise = 1e-4 * torch.randn(ny, nx, generator=g, device="cuda", dtype=torch.float64)
    if flow == "shear":
        return 0.1 + 0.05 * torch.sin(2 * math.pi * y) + noise, 0.02 * torch.sin(2 * math.pi * x) + noise
    band = torch.where(y <= 0.5, torch.tanh(80 * (y - 0.25)), torch.tanh(80 * (0.75 - y)))
    return 0.04 * band + 0.0 * x, 0.002 * torch.sin(2 * math.pi * x) + noise


@pytest.mark.parametrize("pattern", ["ab", "aa"])
@pytest.mark.parametrize("model", ["bgk", "partial", "complete"])
@pytest.mark.parametrize("flow", ["shear", "layer"])
def test_fp32_gradient_has_no_bias(flow, model, pattern):
    """Gradient of the final kinetic energy after 400 steps of a smooth flow. Each reverse step
    rounds nine values per node to half a unit roundoff (2^-24) and the flow's diffusion averages
    such errors away, so the relative error stays at a few roundoffs however many steps there are,
    unless rounding is biased, which adds up over the steps: at most 8 roundoffs in the root mean
    square."""
    import torch
    from paper_2602_21242_amd import LBMFunction
    nx, ny, steps = 333, 190, 400
    ux, uy = (a.float().double() for a in _fields(flow, nx, ny))
    grads = []
    for storage, t in (("f64", torch.float64), ("f32", torch.float32)):
        a, b = ux.to(t).requires_grad_(True), uy.to(t).requires_grad_(True)
        rho, vx, vy = LBMFunction.apply(a, b, dict(nx=nx, ny=ny, theta=1 / 3, nu=0.02, steps=steps, model=model,
                                                   storage=storage, pattern=pattern))
        energy = (0.5 * rho * (vx * vx + vy * vy)).sum()
        grads.append(torch.stack([u.double() for u in torch.autograd.grad(energy, (a, b))]))
    err = float((grads[1] - grads[0]).norm() / grads[0].norm())
    print(f"{flow} {model} {pattern}: rms error {err:.2e}")
    assert err <= 8 * 2.0 ** -24
