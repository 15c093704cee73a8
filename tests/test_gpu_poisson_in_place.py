"""vl_poisson with E in the memory of the moments it reads: the same field as
with an E of its own.  120000 cells are more blocks than run at once."""
import numpy as np
import pytest

from gpu_util import dev, ensure_lib
from paper_2109_06743_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,at", [(64, 0), (257, 0), (257, 300), (257, 771), (120000, 0)])
def test_in_place(nx, at):
    import torch
    from paper_2109_06743_amd import vl
    ensure_lib()
    cfg, _ = W.landau(nx=nx, nv=8)
    ctx = vl.Context(cfg, "f64")
    mom = dev(1.0 + 0.1 * np.random.default_rng(nx).normal(size=(nx, 4)), "f64")
    apart = torch.zeros(nx, dtype=torch.float64, device="cuda")
    ctx.poisson(mom, apart)
    rest = mom.clone()
    E = mom[at:at + nx]
    ctx.poisson(mom, E)
    ctx.sync()
    assert torch.equal(E, apart)
    rest[at:at + nx] = apart
    assert torch.equal(mom, rest)
