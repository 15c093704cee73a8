"""Weight gradient of the heat-flux network where its launch changes form: one
row, fewer than four tiles of 16 rows in a block, several rounds of four, a last
round that is not full, and counts of block sums around whole rounds of 64."""
import numpy as np
import pytest

from gpu_util import ensure_lib, host, rel_l2
from oracle import mlp as OM
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def lib():
    ensure_lib()


@pytest.mark.parametrize("n", [1, 17, 16 * 63, 16 * 64 + 1, 16 * 191 + 3, 16 * 256, 16 * 256 + 1, 16 * 769, 16 * 1024,
                               16 * 1025 - 7, 16 * 2049])
def test_gradient(n):
    """Against the oracle with the tolerance of the other gradient tests.  A few
    rows -- the first, the last, those about the edges of the first tiles -- carry
    targets sqrt(n) times the others, so that leaving one out would show."""
    import torch
    from paper_2109_06743_amd import vl
    ctx = vl.Context(dict(W.gem(nx=4, ny=2, nv=8)[0]), "f32")
    rng = np.random.default_rng(n)
    x = torch.as_tensor(rng.normal(size=(n, 64)).astype(np.float32)).to(torch.bfloat16)
    t = np.zeros((n, 16), dtype=np.float32)
    t[:, :10] = rng.normal(scale=0.5, size=(n, 10))
    heavy = [r for r in (0, 15, 16, 47, 48, 63, 64, 79, n - 17, n - 1) if 0 <= r < n]
    t[heavy] *= np.sqrt(n)
    p = W.mlp_init(3)
    work = torch.zeros(ctx.mlp_work_size(n), dtype=torch.float32, device="cuda")
    gl = torch.zeros(OM.N_PARAM + 1, dtype=torch.float32, device="cuda")
    ctx.mlp_gradient(torch.as_tensor(np.asarray(p, dtype=np.float32)).cuda(), x.view(torch.int16).cuda(),
                     torch.as_tensor(t).cuda(), work, gl)
    ctx.sync()
    L, g = OM.gradient(np.asarray(p), x.double().numpy(), t.astype(np.float64))
    got = host(gl)
    assert abs(got[-1] - L) / L < 1e-2
    for name, off, shape in OM._LAYOUT:
        size = int(np.prod(shape))
        assert rel_l2(got[off:off + size], g[off:off + size]) < 2e-2, name
