"""The maximum of f that one step keeps for the next, beyond what the 2X3V
fitting steps of test_gpu_maxima cover: steps without fitting, where the last X
sweep leaves it, 1X1V steps on both sides of 1024 cells, where the kernels'
partial maxima stop fitting the slot, and steps of another dt, whose X sweep
leaves another number of them, around and inside a graph."""
import numpy as np
import pytest

from gpu_util import ensure_lib
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


def _state(cfg, f, fields, dtype):
    from paper_2109_06743_amd import vl
    ctx = vl.Context(cfg, dtype)
    return ctx, vl.StepState(ctx, f, fields)


def _same(a, b):
    import torch
    for name in ("f", "mom_post"):
        for x, y in zip(getattr(a, name), getattr(b, name)):
            assert torch.equal(x, y), name
    assert torch.equal(a.fields, b.fields)


def _kept_and_recomputed(cfg, f, fields, dtype):
    runs = []
    for recompute in (False, True):
        ctx, st = _state(cfg, f, fields, dtype)
        for _ in range(3):
            if recompute:
                st.c.f_max_valid = 0
            ctx.step(st, cfg["dt"])
        ctx.sync()
        runs.append(st)
    _same(*runs)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny,nv", [(8, 8, 8), (13, 5, 8), (41, 25, 8), (3, 2, 34), (65, 64, 12)])
def test_without_fitting(nx, ny, nv, dtype):
    from paper_2109_06743_amd import vl
    cfg, f, F0 = W.gem(nx=nx, ny=ny, nv=nv, dt=0.001, fit=False, dtype=np.float64)
    _kept_and_recomputed(cfg, f, vl.yee_pack(F0), dtype)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("fit", [True, False])
@pytest.mark.parametrize("nx", [64, 65, 1024, 1025, 3000])
def test_line(nx, fit, dtype):
    cfg, f = W.twostream(nx=nx, nv=40, fit=fit)
    cfg["dt"] = 0.4 * (cfg["x_hi"] - cfg["x_lo"]) / nx / cfg["v_hi"]
    _kept_and_recomputed(cfg, [f], np.zeros(nx), dtype)


def _wide_grid():
    """24800 x 16 cells of 2^3: one y segment (775 blocks, whose maxima the
    next step's waves fold) for shifts beyond a cell, two (1550, folded by a
    launch) below."""
    from paper_2109_06743_amd import vl
    cfg, f, F0 = W.gem(nx=24800, ny=16, nv=2, fit=False, dtype=np.float64)
    cfg.update(x_lo=0.0, x_hi=24800.0, c=1.0)
    dy = (cfg["y_hi"] - cfg["y_lo"]) / 16
    cell = 2.0 * dy / cfg["species"][0]["v_hi"][1]          # the dt whose half step moves the fastest cell by one
    return cfg, f, vl.yee_pack(F0), 0.6 * cell, 1.2 * cell


def test_graph_of_another_dt():
    """A step of dt2 captured after an eager one of dt1 and replayed, against
    the same steps run eagerly."""
    import torch
    cfg, f, fields, dt1, dt2 = _wide_grid()
    (ca, sa), (cb, sb) = _state(cfg, f, fields, "f32"), _state(cfg, f, fields, "f32")
    ca.step(sa, dt1)
    cb.step(sb, dt1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream()):
        cb.step(sb, dt2)                     # recorded, not run
    torch.cuda.synchronize()
    for _ in range(3):
        g.replay()
        ca.step(sa, dt2)
        torch.cuda.synchronize()
        _same(sa, sb)


def test_eager_around_a_graph():
    """Eager steps of dt1 before and after a step of dt2 that is captured and
    replayed once, or never."""
    import torch
    cfg, f, fields, dt1, dt2 = _wide_grid()
    for replays in (0, 1):
        (ca, sa), (cb, sb) = _state(cfg, f, fields, "f32"), _state(cfg, f, fields, "f32")
        for _ in range(2):
            ca.step(sa, dt1)
            cb.step(sb, dt1)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.Stream()):
            cb.step(sb, dt2)
        torch.cuda.synchronize()
        for _ in range(replays):
            g.replay()
            ca.step(sa, dt2)
        torch.cuda.synchronize()
        for _ in range(2):
            ca.step(sa, dt1)
            cb.step(sb, dt1)
        torch.cuda.synchronize()
        _same(sa, sb)
