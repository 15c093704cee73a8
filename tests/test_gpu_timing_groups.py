"""Launch groups that vl_timing_read counts in a step and in single calls."""
import numpy as np
import pytest

from gpu_util import ensure_lib
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("species", [1, 2])
def test_groups(species):
    import torch
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, f, F0 = W.gem(nx=6, ny=4, nv=8, dt=0.001, fit=True, dtype=np.float64)
    cfg["species"] = cfg["species"][:species]
    ctx = vl.Context(cfg, "f32")
    st = vl.StepState(ctx, f[:species], vl.yee_pack(F0))
    ctx.step(st, cfg["dt"])
    ctx.sync()
    ctx.timing_enable(True)
    for _ in range(3):
        ctx.step(st, cfg["dt"])
    ctx.sync()
    got = {k: n for k, (_, n) in ctx.timing_read().items()}
    want = dict(max=0, pfc_x=2, pfc_y=0, pfc_v=1, moments=1, fit=1, copy=0)
    assert {k: got[k] for k in want} == {k: 3 * species * n for k, n in want.items()}
    assert got["fluid"] == 3 and got["fields"] == 6
    cnt = torch.zeros(2, dtype=torch.int64, device="cuda")
    ctx.moment_fit(0, st.f[0], st.f_tmp[0], st.mom_pre[0], st.U[0], counters=cnt)
    ctx.sync()
    assert ctx.timing_read()["fit"][1] == 1
