"""The fused Yee half step (inside the steps) at the edges of its 32 x 8 tiles:
a fluid-model step against the oracle, fields to 1e-13 of the largest one, on
rough fields, between walls and periodic."""
import numpy as np
import pytest

from gpu_util import ensure_lib, host
from oracle import fields as OF, step as OS
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


@pytest.mark.parametrize("bc", ["reflect", "periodic"])
@pytest.mark.parametrize("nx,ny", [(1, 2), (2, 7), (31, 8), (32, 9), (33, 15), (64, 16), (65, 23)])
def test_half_steps(nx, ny, bc):
    from paper_2109_06743_amd import vl
    cfg, U, _ = W.gem_fluid(nx=nx, ny=ny)
    cfg["bc_y"] = bc
    h = min((cfg["x_hi"] - cfg["x_lo"]) / nx, (cfg["y_hi"] - cfg["y_lo"]) / ny)
    dt = 0.2 * h / cfg["c"]
    rng = np.random.default_rng(100 * nx + ny)
    F = OF.Yee(nx, ny)
    for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz"):
        a = 0.05 * rng.normal(size=getattr(F, k).shape)
        if bc == "periodic" and a.shape[0] == ny + 1:
            a[-1] = a[0]
        setattr(F, k, a)
    U = [u * (1 + 0.02 * rng.uniform(-1, 1, size=u.shape[:2] + (1,))) for u in U]
    ctx = vl.Context(cfg, "f64")
    fs = vl.FluidState(ctx, U, vl.yee_pack(F))
    ref = {"U": U, "F": F}
    for _ in range(2):
        ctx.fluid_closure_step(fs, dt, "gradient")
        ref = OS.fluid_step_2x3v(ref, cfg, dt, "gradient")
    ctx.sync()
    yee = vl.yee_unpack(host(fs.fields), nx, ny)
    top = max(np.abs(getattr(ref["F"], k)).max() for k in yee)
    for k in yee:
        assert np.abs(yee[k] - getattr(ref["F"], k)).max() <= 1e-13 * max(top, 1.0), k
