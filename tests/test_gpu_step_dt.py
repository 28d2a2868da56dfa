"""The time step that wm_step forms from its first stage's sweeps, on both sides
of the line (a few thousand signal speeds) between the update that reduces them
and the two kernels that reduce them first."""
import math

import pytest
import torch

from paper_1812_04278_amd import binding as B
from helpers import fields
from test_gpu_parity import gpu_patch

pytestmark = pytest.mark.gpu

CASES = [
    ("fp64", (32, 32, 32), dict()),                                    # 1,536 signal speeds
    ("fp64", (48, 40, 36), dict()),                                    # 3,404
    ("fp64", (43, 43, 43), dict()),                                    # 4,056
    ("fp64", (45, 45, 45), dict()),                                    # 4,860
    ("fp64", (67, 61, 65), dict()),                                    # 13,360
    ("mixed", (67, 61, 65), dict(precision=B.WM_MIXED)),
    ("f32state", (67, 61, 65), dict(precision=B.WM_MIXED_F32STATE)),
    ("rk4-wenoz", (67, 61, 65), dict(integrator=B.WM_RK4, weights=B.WM_WENO_Z)),
    ("walls", (62, 59, 60), dict(walls=(1, 0, 1))),
    ("thin", (8, 8, 400), dict()),
    ("thin-rows", (256, 16, 16), dict()),                              # 3,368
    ("thin-rows", (256, 24, 16), dict()),                              # 4,932
    ("thin-f32", (1, 2, 8192), dict(precision=B.WM_MIXED_F32STATE)),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


def set_thin(p, shape):
    """A state of a box with axes too short, or too long, for the random fields."""
    nx, ny, nz = shape
    x = torch.arange(nx * ny * nz, dtype=torch.float64).reshape(nz, ny, nx)
    one = torch.ones_like(x)
    b = torch.stack([0.5 * one, 0.4 * one, 0.3 * one])
    m = torch.stack([0.3 * torch.sin(0.01 * x), 0.2 * torch.cos(0.02 * x), 0.1 * torch.sin(0.03 * x)])
    p.set_state(1.0 + 0.2 * torch.sin(0.05 * x), m, 2.0 + 0.1 * torch.cos(0.04 * x), b)


@pytest.mark.parametrize("name,shape,kw", CASES, ids=[f"{c[0]}-{'x'.join(map(str, c[1]))}" for c in CASES])
def test_step_dt_bitwise(name, shape, kw):
    """dt and the state after the step are bitwise those of wm_compute_dt and the stages with its dt."""
    print("step dt", name, shape, flush=True)
    pair = []
    for _ in range(2):
        if name.startswith("thin"):
            p = B.Patch(B.config(nx=shape[0], ny=shape[1], nz=shape[2], h=0.01, **kw))
            set_thin(p, shape)
        else:
            p = gpu_patch(fields(max(shape), seed=12, v_rms=1.0, crop=shape), **kw)
        pair.append(p)
    a, b = pair
    for n in range(2):
        dt_b = b.compute_dt()
        b.step_dt(dt_b)
        dt_a = a.step(want_dt=True)
        assert math.isfinite(dt_a) and dt_a > 0.0
        assert dt_a == dt_b, (name, n, dt_a, dt_b)
        sa, sb = a.state(), b.state()
        for k in ("rho", "m", "E", "b"):
            assert torch.equal(sa[k], sb[k]), (name, n, k)


@pytest.mark.parametrize("damage", ["zero_energy", "nan_density", "infinite_energy", "all_negative"])
@pytest.mark.parametrize("shape", [(16, 16, 16), (48, 48, 48)])
def test_step_dt_damaged_state(shape, damage):
    """Failure semantics of both routes: the dt of wm_compute_dt, or NaN on both sides."""
    print("step dt", shape, damage, flush=True)
    f = fields(max(shape), seed=3, v_rms=0.3, kmax=2)
    pa, pb = gpu_patch(f), gpu_patch(f)
    st = pa.state()
    rho, E = st["rho"].clone(), st["E"].clone()
    if damage == "zero_energy":
        E[3, 4, 5] = 0.0
    elif damage == "nan_density":
        rho[7, 8, 9] = float("nan")
    elif damage == "infinite_energy":
        E[2, 2, 2] = float("inf")
    else:
        E.fill_(-50.0)
    for p in (pa, pb):
        p.set_state(rho, st["m"], E, st["b"])
    dt_b = pb.compute_dt()
    dt_a = pa.step(want_dt=True)
    if damage == "nan_density":
        assert math.isnan(dt_a) and math.isnan(dt_b)
    assert dt_a == dt_b or (math.isnan(dt_a) and math.isnan(dt_b)), (dt_a, dt_b)
