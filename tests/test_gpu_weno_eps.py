"""The Jiang-Shu weights at the ends of eps and of the state's magnitude: with
differences that vanish exactly, the weights are formed from powers of eps
alone, and products of them must stay in the range of the work type."""
import dataclasses

import pytest
import torch

from oracle import mhd
from paper_1812_04278_amd import binding as B
from helpers import assert_state_parity, state_errors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


def slabs(nx=40, ny=6, nz=5):
    """Two uniform slabs along x: equal zones but for the two jumps."""
    left = (torch.arange(nx) < nx // 2).double().expand(nz, ny, nx)
    mix = lambda l, r: l * left + r * (1.0 - left)
    rho = mix(1.0, 0.6)
    v = torch.stack([mix(0.2, 0.1), mix(-0.1, 0.3), mix(0.3, 0.0)])
    b = torch.stack([0.75 + 0.0 * left, mix(0.5, -0.25), mix(0.25, 0.5)])
    E = mix(1.0, 0.5) + 0.5 * rho * (v * v).sum(0) + 0.5 * (b * b).sum(0)
    return dict(rho=rho, m=rho * v, E=E, b=b), mhd.Config(nx, ny, nz, 1.0 / nx)


# the smallest eps whose fourth power, and in FP32 second power, is a number of the work
# type, the next decades, and both sides of the line between the two forms of the weights
@pytest.mark.parametrize("precision,eps,tol", [
    (B.WM_FP64, 1e-76, 1e-12), (B.WM_FP64, 1e-75, 1e-12), (B.WM_FP64, 9e-71, 1e-12), (B.WM_FP64, 1.1e-70, 1e-12),
    (B.WM_MIXED_F32STATE, 5e-18, 5e-6), (B.WM_MIXED_F32STATE, 9e-17, 5e-6), (B.WM_MIXED_F32STATE, 1.1e-16, 5e-6)])
def test_step_smallest_eps(precision, eps, tol):
    print("eps", precision, eps, flush=True)
    U, cfg = slabs()
    cfg = dataclasses.replace(cfg, eps=eps)
    p = B.Patch(B.config(nx=cfg.nx, ny=cfg.ny, nz=cfg.nz, h=cfg.h, eps=eps, precision=precision))
    p.set_state(U["rho"], U["m"], U["E"], U["b"])
    U1, dt = mhd.step(U, cfg)
    dt_g = p.step(want_dt=True)
    assert abs(dt_g - dt) <= max(tol, 1e-14) * dt
    if precision == B.WM_FP64:
        assert_state_parity(p.state(), U1, tol, label=str(eps))
    else:
        assert max(state_errors(p.state(), U1).values()) <= tol
