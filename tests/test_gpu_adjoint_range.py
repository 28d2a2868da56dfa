"""The Jiang-Shu weights' gradient at the ends of eps and of the state's
magnitude, where products of the smoothness indicators leave the FP64 range first."""
import pytest
import torch

from oracle import mhd
from paper_1812_04278_amd import binding as B
from helpers import fields, oracle_state
from test_gpu_adjoint import TOL, check8, oracle_vjp, to_gpu_state

pytestmark = pytest.mark.gpu

SHAPE = (12, 10, 9)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


def lam_of(U, seed):
    return torch.randn((8,) + U["rho"].shape, generator=torch.Generator().manual_seed(seed), dtype=torch.float64)


def patch(eps, h):   # eps_B, an absolute bound, below every |B_t|^2 here
    nx, ny, nz = SHAPE
    return B.Patch(B.config(nx=nx, ny=ny, nz=nz, h=h, eps=eps, eps_B=1e-80))


# equal zones: the weights are the linear ones and their gradient vanishes for every
# eps; the smallest whose cube FP64 holds, and both sides of the line between the forms
@pytest.mark.parametrize("eps", [1e-102, 1e-80, 1e-60, 0.9e-50, 1.1e-50, 1e-6])
def test_rhs_vjp_equal_zones(eps):
    print("adjoint, equal zones, eps", eps, flush=True)
    nx, ny, nz = SHAPE
    one = torch.ones((nz, ny, nx), dtype=torch.float64)
    v, b = (0.2, -0.1, 0.3), (0.75, 0.5, -0.25)
    U = dict(rho=0.8 * one, m=torch.stack([0.8 * x * one for x in v]), E=1.7 * one, b=torch.stack([x * one for x in b]))
    cfg = mhd.Config(nx, ny, nz, 0.1)
    lam = lam_of(U, 4)
    h, bf = to_gpu_state(U)
    check8(patch(eps, cfg.h).rhs_vjp(h, bf, lam.cuda()).cpu(), oracle_vjp(lambda X: mhd.rhs(X, cfg), U, lam), str(eps))


# (rho, m, E, b, eps) -> (S rho, S m, S E, sqrt(S) b, S^2 eps) carries the hydro fluxes by S and
# the field's by sqrt(S).  S is a power of four, so no operation rounds otherwise.
@pytest.mark.parametrize("log2", [-150, -60, 60, 150])
def test_rhs_vjp_magnitude(log2):
    print("adjoint, magnitude 2 **", log2, flush=True)
    U, cfg = oracle_state(fields(12, seed=5, v_rms=0.8, crop=SHAPE), h=0.1)
    lam = lam_of(U, 6).cuda()
    h, b = to_gpu_state(U)
    S, R = 2.0 ** log2, 2.0 ** (log2 // 2)
    ref = patch(1e-6, cfg.h).rhs_vjp(h, b, lam)
    lam[5:] *= R
    out = patch(1e-6 * S * S, cfg.h).rhs_vjp(S * h, R * b, lam)
    out[5:] /= R
    check8(out.cpu(), ref.cpu(), f"2^{log2}", TOL)
