"""The adjoint sweep's run-time tiles and launch classes against autograd
through the oracle, at the axis lengths where they can go wrong: the shortest
axes (a tile longer than the axis, several of its positions on one zone), one
tile that spans the axis and wraps onto itself, at and past the longest tile
(256 faces), a short last tile, several whole columns to a wave, and column
counts no tile divides."""
import dataclasses

import pytest
import torch

from oracle import mhd
from paper_1812_04278_amd import binding as B
from helpers import fields, oracle_state
from test_gpu_adjoint import check8, conditioning_tol, oracle_vjp, to_gpu_state

pytestmark = pytest.mark.gpu

SIZES = [(3, 4, 5), (5, 3, 6), (13, 7, 3), (60, 5, 4), (64, 5, 3), (5, 66, 3), (4, 3, 67), (131, 3, 4), (3, 257, 4), (256, 3, 3),
         (262, 4, 3), (3, 5, 259), (16, 32, 8), (8, 33, 16)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


@pytest.mark.parametrize("shape", SIZES)
def test_rhs_vjp_tile_sizes(shape):
    print("adjoint tiles", shape, flush=True)
    n = max(max(shape), 8)
    U, cfg = oracle_state(fields(n + n % 2, seed=21, v_rms=0.8, kmax=2 if n < 64 else 4, crop=shape), h=0.1)
    g = torch.Generator().manual_seed(8)
    lam = torch.randn((8,) + U["rho"].shape, generator=g, dtype=torch.float64)
    fn = lambda X: mhd.rhs(X, cfg)
    ref = oracle_vjp(fn, U, lam)
    p = B.Patch(B.config(nx=cfg.nx, ny=cfg.ny, nz=cfg.nz, h=cfg.h))
    h, b = to_gpu_state(U)
    out = p.rhs_vjp(h, b, lam.cuda())
    check8(out.cpu(), ref, str(shape), conditioning_tol(fn, U, lam, ref))
    assert torch.equal(out, p.rhs_vjp(h, b, lam.cuda()))   # fixed order of the additions


# one launch of the three sweeps: tiles that span all axes, WENO-Z; the last has two tiles on z
@pytest.mark.parametrize("shape", [(3, 3, 3), (17, 33, 9), (64, 9, 70), (9, 4, 300)])
def test_rhs_vjp_weno_z_one_launch(shape):
    print("adjoint, one launch", shape, flush=True)
    n = max(max(shape), 8)
    U, cfg = oracle_state(fields(n + n % 2, seed=5, v_rms=0.8, kmax=2 if n < 64 else 4, crop=shape), h=0.1)
    cfg = dataclasses.replace(cfg, weights="z")
    g = torch.Generator().manual_seed(9)
    lam = torch.randn((8,) + U["rho"].shape, generator=g, dtype=torch.float64)
    fn = lambda X: mhd.rhs(X, cfg)
    ref = oracle_vjp(fn, U, lam)
    p = B.Patch(B.config(nx=cfg.nx, ny=cfg.ny, nz=cfg.nz, h=cfg.h, weights=B.WM_WENO_Z))
    h, b = to_gpu_state(U)
    for _ in range(3):   # the arrays of the y and z sweeps are stored into, not added to
        check8(p.rhs_vjp(h, b, lam.cuda()).cpu(), ref, str(shape), conditioning_tol(fn, U, lam, ref))
