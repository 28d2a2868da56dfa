"""The adjoint's one launch for three sweeps against separate launches: a periodic
box doubled along an axis has the doubled cotangents, and passes the size up to
which the sweeps go together."""
import pytest
import torch

from paper_1812_04278_amd import binding as B
from helpers import fields, oracle_state, rel_err
from test_gpu_adjoint import to_gpu_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


# 265,980 zones (one launch) and 531,960 (separate); the doubled axis is one tile in both
@pytest.mark.parametrize("weights", [B.WM_WENO_JS, B.WM_WENO_Z])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_rhs_vjp_doubled_box(axis, weights):
    shape = {0: (62, 66, 65), 1: (66, 62, 65), 2: (66, 65, 62)}[axis]
    print("adjoint, doubled box", shape, axis, flush=True)
    U, cfg = oracle_state(fields(66, seed=7, v_rms=0.8, crop=shape), h=0.1)
    h, b = to_gpu_state(U)
    lam = torch.randn((8,) + tuple(U["rho"].shape), generator=torch.Generator().manual_seed(2), dtype=torch.float64).cuda()

    def vjp(n, *t):
        return B.Patch(B.config(nx=n[0], ny=n[1], nz=n[2], h=cfg.h, weights=weights)).rhs_vjp(*t)

    twice = lambda x: torch.cat([x, x], dim=3 - axis)
    ref = twice(vjp(shape, h, b, lam))
    big = tuple(s * (2 if d == axis else 1) for d, s in enumerate(shape))
    out = vjp(big, twice(h), twice(b), twice(lam))
    # the same terms of a zone's cotangent in another order of addition
    assert max(rel_err(out[c], ref[c]) for c in range(8)) <= 1e-12
