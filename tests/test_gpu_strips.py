"""X(tau) of 2X3V on both sides of the line between narrow (4 columns, segments
down to 4 rows) and wide (8 columns) strips of cells: the last grid that takes
the narrow ones, the next one, short segments, strips and segments that are not
full, shifts below a cell and of several cells, both y boundaries."""
import numpy as np
import pytest

from gpu_util import TOL_SWEEP, dev, ensure_lib, host, rel_l2, storage_round
from oracle import step as OS, vlasov as OV
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bc", ["reflect", "periodic"])
@pytest.mark.parametrize("nx,ny,nv,cells", [(128, 128, 8, 0.7), (129, 128, 8, 0.7), (129, 121, 8, 2.6), (5, 3, 8, 0.9),
                                            (9, 23, 8, 0.4), (33, 22, 6, 3.3), (4, 13, 12, 1.2), (310, 16, 12, 0.8)])
def test_x_operator(nx, ny, nv, cells, bc, dtype):
    import torch
    from paper_2109_06743_amd import vl
    cfg = (W.gem(nx=nx, ny=ny, nv=2, dtype=np.float64) if bc == "reflect"
           else W.orszag_tang(n=nx, ny=ny, nv=2, dtype=np.float64))[0]
    cfg["species"] = [dict(sp, nv=[nv] * 3) for sp in cfg["species"]]
    dx = (cfg["x_hi"] - cfg["x_lo"]) / nx
    dy = (cfg["y_hi"] - cfg["y_lo"]) / ny
    sp = cfg["species"][0]
    v, _ = OS._grids(cfg, sp)
    tau = cells * min(dx, dy) / max(np.abs(v[0]).max(), np.abs(v[1]).max())
    f = storage_round(W.random_block((ny, nx, nv, nv, nv), seed=nx + ny, kind="smooth"), dtype)
    ctx = vl.Context(cfg, dtype)
    fin = dev(f, dtype)
    out = torch.empty_like(fin)
    ctx.pfc_advect_x(0, fin, out, tau)
    ctx.sync()
    ref = OV.x_advect_2x3v(f, v[0], v[1], dx, dy, tau, f_inf=float(f.max()), bc_y=bc)
    got = host(out, ref.shape)
    assert rel_l2(got, ref) < (TOL_SWEEP[dtype] if bc == "reflect" else 2 * TOL_SWEEP[dtype])
    assert abs(got.sum() - f.sum()) <= (1e-6 if dtype == "f32" else 1e-12) * f.sum()
