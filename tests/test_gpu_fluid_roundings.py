"""The fluid step to the last bit.  The fit rounds functions of U to FP32
coefficients of the distribution, so a last bit of U can become one of f; the
kernels' roundings are therefore fixed, and these tests form the same on the
host (fluid_roundings) and allow no difference."""
import numpy as np
import pytest

import fluid_roundings as FR
from gpu_util import dev, ensure_lib, host, rel_l2
from oracle import fields as OF, fluid as OFL
from paper_2109_06743_amd import workloads as W


def _kinetic(nx, ny, bc, s):
    cfg, U0, _ = W.gem_fluid(nx=nx, ny=ny)
    cfg["bc_y"] = bc
    rng = np.random.default_rng(nx * 100 + ny + s)
    mom = [np.concatenate([U0[s], 0.1 * rng.normal(size=(ny, nx, 10))], axis=-1)
           * (1 + 0.1 * rng.uniform(-1, 1, size=(ny, nx, 20))) for _ in range(2)]
    U = U0[s] * (1 + 0.1 * rng.uniform(-1, 1, size=(ny, nx, 10)))
    U[..., 1:4] += 0.1 * U[..., :1] * rng.normal(size=(ny, nx, 3))
    fl = [rng.normal(scale=0.3, size=(ny, nx, 3)) for _ in range(6)]
    dx, dy = (cfg["x_hi"] - cfg["x_lo"]) / nx, (cfg["y_hi"] - cfg["y_lo"]) / ny
    return cfg, cfg["species"][s], U, mom, fl, dx, dy, 0.01 * min(dx, dy)


def _kinetic_ref(sp, U, mom, fl, dx, dy, dt, bc):
    Q = [mom[0][..., 10:], mom[1][..., 10:], 0.5 * mom[0][..., 10:] + 0.5 * mom[1][..., 10:]]
    return FR.rk3_3v(U, lambda k, _: Q[k], [(fl[2 * k], fl[2 * k + 1]) for k in range(3)], sp["q"], sp["m"], dx, dy,
                     dt, bc)


def test_fma():
    """The host's fma rounds exactly: against rationals."""
    from fractions import Fraction
    rng = np.random.default_rng(0)
    a, b = rng.normal(size=400), rng.normal(size=400)
    c = np.where(rng.random(400) < 0.5, -a * b * (1 + rng.integers(-3, 4, 400) * 2.0 ** -52), rng.normal(size=400))
    got = FR.fma(a, b, c)
    for x, y, z, g in zip(a, b, c, got):
        assert g == float(Fraction(x) * Fraction(y) + Fraction(z))


@pytest.mark.parametrize("bc", ["reflect", "periodic"])
def test_host_stage_is_the_oracles(bc):
    """The host form computes what the oracle does, to rounding."""
    cfg, sp, U, mom, fl, dx, dy, dt = _kinetic(9, 7, bc, 1)
    ref = OFL.rk3_3v(U, mom[0][..., 10:], mom[1][..., 10:], *[(fl[2 * k], fl[2 * k + 1]) for k in range(3)], sp["q"],
                     sp["m"], dx, dy, dt, bc)
    assert rel_l2(_kinetic_ref(sp, U, mom, fl, dx, dy, dt, bc), ref) < 1e-14


@pytest.mark.gpu
@pytest.mark.parametrize("bc", ["reflect", "periodic"])
@pytest.mark.parametrize("s", [0, 1])
@pytest.mark.parametrize("nx,ny", [(1, 2), (15, 17), (43, 48)])
def test_kinetic(nx, ny, s, bc):
    import torch
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, sp, U, mom, fl, dx, dy, dt = _kinetic(nx, ny, bc, s)
    ctx = vl.Context(cfg, "f64")
    Ud = dev(U, "f64")
    work = torch.empty(ctx.fluid_work_size(), dtype=torch.float64, device="cuda")
    ctx.fluid_step(s, Ud, dev(mom[0], "f64"), dev(mom[1], "f64"), *[dev(a, "f64") for a in fl], dt, work)
    ctx.sync()
    np.testing.assert_array_equal(host(Ud, U.shape), _kinetic_ref(sp, U, mom, fl, dx, dy, dt, bc))


@pytest.mark.gpu
@pytest.mark.parametrize("closure,nx,ny", [("gradient", 15, 17), ("gradient", 43, 48), ("mlp", 1, 2), ("mlp", 15, 17),
                                           ("mlp", 63, 3), ("mlp", 64, 4), ("mlp", 65, 5), ("mlp", 129, 9)])
def test_closures(closure, nx, ny):
    """Both species of a fluid-model step; the stage fields and the network's
    outputs are the library's own (of the separate features and forward calls;
    the step has both in one kernel of 64 x 4 tiles), the rest is formed on the
    host.  The network adds 1e-5 of U and less, a billion times what would show."""
    import torch
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, U, F0 = W.gem_fluid(nx=nx, ny=ny, dt=0.003)
    rng = np.random.default_rng(nx * 100 + ny)
    U = [u * (1 + 0.05 * rng.uniform(-1, 1, size=u.shape)) for u in U]
    F = OF.Yee(nx, ny)
    for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz"):
        setattr(F, k, getattr(F0, k).copy())
    dx, dy, dt = (cfg["x_hi"] - cfg["x_lo"]) / nx, (cfg["y_hi"] - cfg["y_lo"]) / ny, cfg["dt"]
    net = W.mlp_init(3)
    ctx = vl.Context(cfg, "f64")
    fs = vl.FluidState(ctx, U, vl.yee_pack(F), mlp_params=net)
    ctx.fluid_closure_step(fs, dt, closure)

    def zeros():
        return torch.zeros(nx * ny * 3, dtype=torch.float64, device="cuda")
    yee, eb = dev(vl.yee_pack(F), "f64"), [zeros() for _ in range(4)]
    ctx.cell_fields(yee, eb[0], eb[1])
    ctx.maxwell_half_step(yee, [dev(np.concatenate([u, np.zeros_like(u)], -1), "f64") for u in U], dt)
    ctx.cell_fields(yee, eb[2], eb[3])
    ctx.sync()
    E_t, B_t, E_h, B_h = [host(x, (ny, nx, 3)) for x in eb]
    fields = [(E_t, B_t), (2.0 * E_h - E_t, 2.0 * B_h - B_t), (E_h, B_h)]
    for s, sp in enumerate(cfg["species"]):
        def third(k, V):
            if closure == "gradient":
                return FR.third_moment(V, sp["m"])
            x = torch.zeros((ny * nx, 64), dtype=torch.int16, device="cuda")
            sc = torch.zeros(ny * nx, dtype=torch.float64, device="cuda")
            y = torch.zeros((ny * nx, 16), device="cuda")
            ctx.mlp_features(s, dev(V, "f64"), 10, x, sc, B=dev(fields[k][1], "f64"))
            ctx.mlp_forward(fs.mlp_params, x, y)
            ctx.sync()
            return FR.third_moment(V, sp["m"], host(sc, (ny, nx)), host(y, (ny, nx, 16)))
        ref = FR.rk3_3v(U[s], third, fields, sp["q"], sp["m"], dx, dy, dt, "reflect",
                        FR.eq5_strength(sp["q"], sp["m"]) if closure == "gradient" else None)
        np.testing.assert_array_equal(host(fs.U[s], U[s].shape), ref, err_msg=f"species {s}")


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(1, 2), (63, 3), (64, 4), (65, 5), (129, 9)])
def test_features_at_tile_edges(nx, ny):
    """The features that test_closures takes as given, against the oracle's: FP64
    values rounded to FP32 and BF16, so at most one BF16 step apart where a
    rounding flips, differences of equal values aside."""
    import torch
    from oracle import mlp as OM
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, U, _ = W.gem_fluid(nx=nx, ny=ny)
    rng = np.random.default_rng(nx * 100 + ny)
    B = rng.normal(size=(ny, nx, 3))
    ctx = vl.Context(cfg, "f64")
    for s, sp in enumerate(cfg["species"]):
        V = U[s] * (1 + 0.05 * rng.uniform(-1, 1, size=U[s].shape))
        x = torch.zeros((ny * nx, 64), dtype=torch.int16, device="cuda")
        sc = torch.zeros(ny * nx, dtype=torch.float64, device="cuda")
        ctx.mlp_features(s, dev(V, "f64"), 10, x, sc, B=dev(B, "f64"))
        ctx.sync()
        rx, rs = OM.features_bf16(V, sp["m"], s, B)
        rx = np.asarray(rx, dtype=np.float64).reshape(ny * nx, 64)
        got = x.view(torch.bfloat16).double().cpu().numpy()
        np.testing.assert_allclose(got, rx, rtol=2.0 ** -7, atol=1e-12)
        assert (np.abs(got - rx) > 1e-12).mean() < 1e-3
        np.testing.assert_allclose(host(sc), np.asarray(rs).reshape(-1), rtol=1e-13)


@pytest.mark.gpu
@pytest.mark.parametrize("nx", [3, 56, 200])
def test_line(nx):
    import torch
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, _ = W.landau(nx=nx, nv=8)
    ctx = vl.Context(cfg, "f64")
    rng = np.random.default_rng(nx)
    U = np.stack([1 + 0.3 * rng.uniform(size=nx), 0.2 * rng.normal(size=nx), 1 + 0.3 * rng.uniform(size=nx)], -1)
    mom = [rng.normal(size=(nx, 4)) for _ in range(2)]
    E = [rng.normal(size=nx) for _ in range(3)]
    dx = (cfg["x_hi"] - cfg["x_lo"]) / nx
    dt = 0.05 * dx
    Ud = dev(U, "f64")
    work = torch.empty(ctx.fluid_work_size(), dtype=torch.float64, device="cuda")
    ed = [dev(e, "f64") for e in E]
    ctx.fluid_step(0, Ud, dev(mom[0], "f64"), dev(mom[1], "f64"), ed[0], None, ed[1], None, ed[2], None, dt, work)
    ctx.sync()
    ref = FR.rk3_1v(U, [mom[0][:, 3], mom[1][:, 3], 0.5 * mom[0][:, 3] + 0.5 * mom[1][:, 3]], E, cfg["q"], cfg["m"],
                    dx, dt)
    np.testing.assert_array_equal(host(Ud, U.shape), ref)
