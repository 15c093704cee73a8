"""The fluid stage kernel at the edges of its 14 x 16 tiles: one cell less, as
many and one more, grids smaller than the two halo cells, walls and periodic
y, with the kinetic third moment and with the Eq. 5 closure."""
import numpy as np
import pytest

from gpu_util import dev, ensure_lib, host, rel_l2
from oracle import fields as OF, fluid as OFL, step as OS
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu
SIZES = [(1, 2), (2, 3), (13, 15), (14, 16), (15, 17), (29, 33), (28, 14), (43, 48)]


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


@pytest.mark.parametrize("bc", ["reflect", "periodic"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_kinetic_stage_tiles(nx, ny, bc):
    """vl_fluid_step against the oracle on rough states (10 % noise): FP64
    rounding in the same formulas, 1e-12."""
    import torch
    from paper_2109_06743_amd import vl
    cfg, U0, _ = W.gem_fluid(nx=nx, ny=ny)
    cfg["bc_y"] = bc
    ctx = vl.Context(cfg, "f64")
    dx, dy = (cfg["x_hi"] - cfg["x_lo"]) / nx, (cfg["y_hi"] - cfg["y_lo"]) / ny
    rng = np.random.default_rng(nx * 100 + ny)
    s, sp = 1, cfg["species"][1]
    mom = [np.concatenate([U0[s], 0.1 * rng.normal(size=(ny, nx, 10))], axis=-1)
           * (1 + 0.1 * rng.uniform(-1, 1, size=(ny, nx, 20))) for _ in range(2)]
    U = U0[s] * (1 + 0.1 * rng.uniform(-1, 1, size=(ny, nx, 10)))
    fl = [rng.normal(scale=0.3, size=(ny, nx, 3)) for _ in range(6)]
    dt = 0.01 * min(dx, dy)
    ref = OFL.rk3_3v(U, mom[0][..., 10:], mom[1][..., 10:], (fl[0], fl[1]), (fl[2], fl[3]), (fl[4], fl[5]),
                     sp["q"], sp["m"], dx, dy, dt, bc)
    Ud = dev(U, "f64")
    work = torch.empty(ctx.fluid_work_size(), dtype=torch.float64, device="cuda")
    ctx.fluid_step(s, Ud, dev(mom[0], "f64"), dev(mom[1], "f64"), *[dev(a, "f64") for a in fl], dt, work)
    ctx.sync()
    np.testing.assert_allclose(host(Ud, ref.shape), ref, rtol=1e-12, atol=1e-13 * np.abs(ref).max())


@pytest.mark.parametrize("bc", ["reflect", "periodic"])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_gradient_stage_tiles(nx, ny, bc):
    """One step of the fluid model with Eq. 5, both species in one launch."""
    from paper_2109_06743_amd import vl
    cfg, U, F0 = W.gem_fluid(nx=nx, ny=ny, dt=1e-4)
    cfg["bc_y"] = bc
    rng = np.random.default_rng(nx * 100 + ny)
    U = [u * (1 + 0.05 * rng.uniform(-1, 1, size=u.shape[:2] + (1,))) for u in U]
    F = OF.Yee(nx, ny)
    for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz"):
        a = getattr(F0, k).copy()
        if bc == "periodic" and a.shape[0] == ny + 1:
            a[-1] = a[0]
        setattr(F, k, a)
    ctx = vl.Context(cfg, "f64")
    fs = vl.FluidState(ctx, U, vl.yee_pack(F))
    ctx.fluid_closure_step(fs, cfg["dt"], "gradient")
    ref = OS.fluid_step_2x3v({"U": [u.copy() for u in U], "F": F}, cfg, cfg["dt"], "gradient")
    ctx.sync()
    for s in range(2):
        assert rel_l2(host(fs.U[s], U[s].shape), ref["U"][s]) < 1e-12, s


@pytest.mark.parametrize("nx,ny", [(1, 2), (63, 3), (64, 4), (65, 5), (129, 9)])
def test_network_tiles(nx, ny):
    """Features and network in one kernel at the edges of its 64 x 4 tiles: a
    step of the fluid model with the network closure, U to 2e-5 (the network
    rounds activations to BF16, the oracle's does not)."""
    from paper_2109_06743_amd import vl
    cfg, U, F0 = W.gem_fluid(nx=nx, ny=ny, dt=1e-4)
    rng = np.random.default_rng(nx * 100 + ny)
    U = [u * (1 + 0.05 * rng.uniform(-1, 1, size=u.shape[:2] + (1,))) for u in U]
    F = OF.Yee(nx, ny)
    for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz"):
        setattr(F, k, getattr(F0, k).copy())
    net = W.mlp_init(3)
    ctx = vl.Context(cfg, "f64")
    fs = vl.FluidState(ctx, U, vl.yee_pack(F), mlp_params=net)
    ctx.fluid_closure_step(fs, cfg["dt"], "mlp")
    ref = OS.fluid_step_2x3v({"U": [u.copy() for u in U], "F": F}, cfg, cfg["dt"], "mlp", net)
    ctx.sync()
    for s in range(2):
        assert rel_l2(host(fs.U[s], U[s].shape), ref["U"][s]) < 2e-5, s
