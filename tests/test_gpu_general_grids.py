"""Velocity grids without a kernel of their own, where the general kernels
change form: every pencil length from 2 to 32 on some axis, shifts below and
beyond a cell in one wave, blocks with few and many pencils, few and many
cells (one or four waves per cell in the moments)."""
import numpy as np
import pytest

from gpu_util import TOL_MOM, dev, ensure_lib, host, rel_l2, storage_round
from oracle import moments as OM, step as OS, vlasov as OV
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu
# together the axes take every length from 2 to 32
GRIDS = [(2, 3, 5), (4, 6, 7), (32, 8, 9), (10, 31, 11), (13, 17, 30), (14, 15, 29), (28, 18, 15), (19, 12, 27),
         (26, 20, 13), (21, 14, 25), (24, 22, 15), (16, 23, 20)]


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


def _problem(nv, dtype, nx=3, ny=2, seed=0):
    cfg, _, _ = W.gem(nx=nx, ny=ny, nv=2, fit=True, dtype=np.float64)
    cfg["species"] = [dict(sp, nv=list(nv)) for sp in cfg["species"]]
    rng = np.random.default_rng(seed + nv[0] * 1024 + nv[1] * 32 + nv[2])
    f = storage_round(np.stack([np.stack([W.random_block(nv, seed + 7 * i + 11 * j + nv[0], "smooth")
                                          for i in range(nx)]) for j in range(ny)]), dtype)
    return cfg, f, rng


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nv", GRIDS)
def test_v_operator(nv, dtype):
    """Five sweeps with shifts from a fraction of a cell to several cells,
    against the oracle per call (the tolerance of the other V tests), mass and
    positivity."""
    from paper_2109_06743_amd import vl
    cfg, f, rng = _problem(nv, dtype)
    s, sp = 0, cfg["species"][0]
    v, dv = OS._grids(cfg, sp)
    tau = 0.01
    # cell 0: sub-cell everywhere; then accelerations of up to four cells
    unit = abs(sp["m"] / sp["q"]) * max(dv) / tau
    E = rng.uniform(-1, 1, size=(2, 3, 3)) * unit * np.linspace(0.3, 4.0, 6).reshape(2, 3, 1)
    B = rng.uniform(-1, 1, size=(2, 3, 3)) * unit / max(sp["v_hi"]) * 0.5
    ctx = vl.Context(cfg, dtype)
    fd = dev(f, dtype)
    out = fd.clone()
    ctx.pfc_advect_v(s, fd, out, dev(E, "f64"), dev(B, "f64"), tau)
    ctx.sync()
    ref = OV.v_advect_3v(f, E, B, sp["q"], sp["m"], v, dv, tau)
    got = host(out, f.shape)
    assert rel_l2(got, ref) < (3e-6 if dtype == "f32" else 3e-13)
    assert (got >= 0).all()
    assert abs(got.sum() - f.sum()) <= (1e-6 if dtype == "f32" else 1e-13) * f.sum()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nv", GRIDS + [(8, 8, 8), (12, 12, 12), (16, 16, 16)])
def test_v_backsub(nv, dtype):
    """The backsubstitution split with feet within a cell of their faces, on
    either side, in the first cell and several cells away in the others (both
    forms in one wave).  FP32: three sweeps, each foot (up to 32 cells) to one
    rounding, slopes of f up to its size per cell."""
    from paper_2109_06743_amd import vl
    cfg, f, rng = _problem(nv, dtype)
    cfg = dict(cfg, vsplit="backsub")
    s, sp = 0, cfg["species"][0]
    v, dv = OS._grids(cfg, sp)
    tau = 0.01
    unit = abs(sp["m"] / sp["q"]) * max(dv) / tau
    E = rng.uniform(-1, 1, size=(2, 3, 3)) * unit * np.linspace(0.3, 4.0, 6).reshape(2, 3, 1)
    B = rng.uniform(-1, 1, size=(2, 3, 3)) * np.linspace(0.2, 4.0, 6).reshape(2, 3, 1)
    ctx = vl.Context(cfg, dtype)
    fd = dev(f, dtype)
    out = fd.clone()
    ctx.pfc_advect_v(s, fd, out, dev(E, "f64"), dev(B, "f64"), tau)
    ctx.sync()
    ref = OV.v_advect_3v_backsub(f, E, B, sp["q"], sp["m"], v, dv, tau)
    got = host(out, f.shape)
    assert rel_l2(got, ref) < (3 * 32 * 2.0 ** -24 if dtype == "f32" else 1e-13)
    assert (got >= 0).all()
    np.testing.assert_allclose(got.sum((2, 3, 4)), f.sum((2, 3, 4)), rtol=1e-6 if dtype == "f32" else 1e-13)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny,nv", [(3, 2, nv) for nv in GRIDS] + [(64, 64, (4, 5, 27)), (63, 65, (3, 12, 11))])
def test_moments_and_fit(nx, ny, nv, dtype):
    """Moments per group and the fit against the oracle on a sample of cells."""
    import torch
    from paper_2109_06743_amd import vl
    cfg, _, _ = W.gem(nx=nx, ny=ny, nv=2, fit=True, dtype=np.float64)
    cfg["species"] = [dict(sp, nv=list(nv)) for sp in cfg["species"]]
    s, sp = 1, cfg["species"][1]
    v, dv = OS._grids(cfg, sp)
    rng = np.random.default_rng(5)
    cells = nx * ny
    base = np.stack([W.random_block(nv, k, "smooth") for k in range(6)])
    f = storage_round(base[np.arange(cells) % 6] * rng.uniform(0.5, 1.5, size=(cells, 1, 1, 1)), dtype)
    ctx = vl.Context(cfg, dtype)
    fd = dev(f, dtype)
    mom = torch.zeros(cells * 20, dtype=torch.float64, device="cuda")
    ctx.moments(s, fd, mom)
    pick = sorted({0, 1, cells // 2, cells - 1})
    ref = OM.raw_moments_3v(f[pick], v, dv, sp["m"])
    got = host(mom, (cells, 20))[pick]
    for lo, hi in ((0, 1), (1, 4), (4, 10), (10, 20)):
        scale = max(np.linalg.norm(ref[:, lo:hi]), 1e-3 * np.linalg.norm(ref[:, 0]))
        assert np.linalg.norm(got[:, lo:hi] - ref[:, lo:hi]) < TOL_MOM[dtype] * scale, lo
    if min(nv) < 4:
        return                                   # too few cells for two temperatures that differ
    U = host(mom, (cells, 20))[:, :10].copy()
    U[:, 4:10:3] *= 1.05
    Ud = dev(U, "f64")
    out, post = torch.zeros_like(fd), torch.zeros_like(mom)
    cnt = torch.zeros(2, dtype=torch.int64, device="cuda")
    ctx.moment_fit(s, fd, out, mom, Ud, post, cnt)
    ctx.sync()
    full = host(out, f.shape)
    for k, c in enumerate(pick):
        g, Uk, _, _ = OM.fit_cell_3v(f[c], ref[k], U[c], sp["m"], v, dv)
        assert rel_l2(full[c], g) < (1e-5 if dtype == "f32" else 1e-12)
        assert rel_l2(host(Ud, U.shape)[c], Uk) < 1e-12
        pk = OM.raw_moments_3v(full[c], v, dv, sp["m"])
        assert rel_l2(host(post, (cells, 20))[c][:10], pk[:10]) < 1e-6
