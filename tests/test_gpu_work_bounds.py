"""The steps stay within the scratch they ask for: a pattern behind it is
untouched, and results do not depend on what the scratch holds or how it is
aligned.  What they ask for is what they use."""
import numpy as np
import pytest

from gpu_util import ensure_lib
from paper_2109_06743_amd import workloads as W

GUARD = 4096


def _guarded(st, n, shift, fill):
    import torch
    buf = torch.full((n + GUARD + 1,), fill, dtype=torch.float64, device="cuda")
    buf[shift + n:] = -7.25
    st.work = buf
    st.c.work = buf[shift:].data_ptr()
    return buf[shift + n:]


def _run(make, step, size):
    import torch
    out = []
    for shift, fill in ((0, 0.0), (0, float("nan")), (1, 3.0)):
        ctx, st = make()
        tail = _guarded(st, size(ctx), shift, fill)
        for _ in range(2):
            step(ctx, st)
        ctx.sync()
        assert bool((tail == -7.25).all())
        out.append([x.clone() for x in list(getattr(st, "f", [])) + list(st.U) + [st.fields]])
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(3, 2), (17, 9)])
@pytest.mark.parametrize("kind", ["fit", "nofit", "network", "backsub"])
def test_step(kind, nx, ny):
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, f, F0 = W.gem(nx=nx, ny=ny, nv=8, fit=kind != "nofit", dtype=np.float64)
    if kind == "network":
        cfg.update(closure="mlp", closure_tol=1e9)
    if kind == "backsub":
        cfg["vsplit"] = "backsub"

    def make():
        ctx = vl.Context(cfg, "f64")
        return ctx, vl.StepState(ctx, f, vl.yee_pack(F0), mlp_params=W.mlp_init(3) if kind == "network" else None)
    _run(make, lambda ctx, st: ctx.step(st, 0.001), lambda ctx: ctx.step_work_size())


@pytest.mark.gpu
@pytest.mark.parametrize("nx", [5, 130])
@pytest.mark.parametrize("fit", [True, False])
def test_line_step(nx, fit):
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, f = W.landau(nx=nx, nv=16, fit=fit)

    def make():
        ctx = vl.Context(cfg, "f64")
        return ctx, vl.StepState(ctx, [f], np.zeros(nx))
    _run(make, lambda ctx, st: ctx.step(st, 0.3 * cfg["dt"]), lambda ctx: ctx.step_work_size())


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(3, 2), (17, 9)])
@pytest.mark.parametrize("closure", ["gradient", "mlp"])
@pytest.mark.parametrize("species", [1, 2])
def test_fluid_closure_step(species, closure, nx, ny):
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, U, F0 = W.gem_fluid(nx=nx, ny=ny, dt=1e-3)
    cfg["species"] = cfg["species"][:species]

    def make():
        ctx = vl.Context(cfg, "f64")
        return ctx, vl.FluidState(ctx, U, vl.yee_pack(F0), mlp_params=W.mlp_init(3))
    _run(make, lambda ctx, st: ctx.fluid_closure_step(st, cfg["dt"], closure), lambda ctx: ctx.fluid_closure_work_size())


def test_sizes():
    """Per cell: fields 18, the Yee arrays between the half steps 6, two stage
    states of 10 per species, the network's 9 per species; 1X1V 7."""
    from paper_2109_06743_amd import vl
    ensure_lib()
    n = 64
    cfg, _, _ = W.gem(nx=n, ny=n, nv=4, fit=True, dtype=np.float64)
    edge = 3 * n + 1024
    assert vl.Context(cfg, "f64").step_work_size() <= (18 + 6 + 40) * n * n + edge
    cfg.update(closure="mlp", closure_tol=0.1)
    ctx = vl.Context(cfg, "f64")
    assert ctx.step_work_size() <= (18 + 6 + 40 + 18) * n * n + edge + 2 * 512
    assert ctx.fluid_closure_work_size() <= (18 + 6 + 40 + 18) * n * n + edge
    assert ctx.fluid_work_size() <= 20 * n * n
    assert vl.Context(W.landau(nx=n, nv=8, fit=True)[0], "f64").step_work_size() <= 7 * n
