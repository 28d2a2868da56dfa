"""The diagnostics and floor-count reductions at the sizes where their index
walk and their trees can go wrong: fewer zones than one block, a single row or
column, sizes that are no multiple of the block, and more zones than one step
of the grid."""
import pytest
import torch

from oracle import mhd
from paper_1812_04278_amd import binding as B
from helpers import assert_diag_parity

pytestmark = pytest.mark.gpu

SIZES = [(7, 1, 1), (1, 1, 300), (1, 17, 19), (255, 3, 2), (67, 61, 65)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


def planted(shape, seed):
    """A random physical state (rho, P > 0, random face field) on a box."""
    g = torch.Generator().manual_seed(seed)
    nx, ny, nz = shape
    r = lambda *s: torch.rand(*s, nz, ny, nx, generator=g, dtype=torch.float64)
    rho, m, b = 0.5 + r(), r(3) - 0.3, r(3) - 0.4
    return dict(rho=rho, m=m, E=4.0 + r(), b=b), mhd.Config(nx, ny, nz, 1.0 / max(shape))


@pytest.mark.parametrize("precision", [B.WM_FP64, B.WM_MIXED_F32STATE])
@pytest.mark.parametrize("shape", SIZES)
def test_diagnostics_sizes(shape, precision):
    print("diagnostics", shape, precision, flush=True)
    U, cfg = planted(shape, 5)
    if precision == B.WM_MIXED_F32STATE:
        U = {k: v.float().double() for k, v in U.items()}
    p = B.Patch(B.config(nx=cfg.nx, ny=cfg.ny, nz=cfg.nz, h=cfg.h, precision=precision))
    p.set_state(U["rho"], U["m"], U["E"], U["b"])
    d, o = p.diagnostics(), mhd.diagnostics(U, cfg)
    if precision == B.WM_MIXED_F32STATE:   # the zone field is stored rounded to 24 bits: P moves by (gamma-1) B dB
        assert abs(d["min_p"] - o["min_p"]) <= (2.0 / 3.0) * 3 * 2.0 ** -24
        o["min_p"] = d["min_p"]
    assert_diag_parity(d, o, U, cfg.h)
    assert p.diagnostics() == d


@pytest.mark.parametrize("shape", SIZES)
def test_floor_count_sizes(shape):
    """dt = 0 leaves the state as it is, so each of the three stage results has
    every planted zone raised once."""
    print("floor count", shape, flush=True)
    U, cfg = planted(shape, 6)
    low = U["rho"] < 0.9
    p = B.Patch(B.config(nx=cfg.nx, ny=cfg.ny, nz=cfg.nz, h=cfg.h, rho_floor=0.9))
    p.set_state(U["rho"], U["m"], U["E"], U["b"])
    p.step_dt(0.0)
    assert p.diagnostics(raise_unphysical=False)["n_floored"] == 3 * int(low.sum())
    assert torch.equal(p.hydro[0].cpu(), U["rho"].clamp(min=0.9))
