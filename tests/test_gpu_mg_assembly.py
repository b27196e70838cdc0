"""The assembled coarse operator is the projected fine one: its nine-point
product equals restrict(D prolong(e)) made of the transfers and the operator
themselves.  Null-vector counts below, at and past the 16 columns of a
matrix-core tile, on lattices of unequal extents."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[False, True])
def case(request):
    return Case((8, 16, 8, 24), 0.3, 0.1355, 1.0, 91, oracle_T=False, antiperiodic_t=request.param)


@pytest.mark.parametrize("nv", [2, 15, 16, 17, 31])
def test_coarse_operator_is_the_projected_operator(case, nv):
    c = case
    etas = c.lat.new_field(cs.F32, nv)
    etas.view(torch.float32).normal_(generator=torch.Generator(device="cuda").manual_seed(92))
    m = cs.Multigrid(c.op, etas, cs.MgParams(nv=nv, n_adapt=0))
    e = torch.randn((m.nblk, m.nc), dtype=torch.complex64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(93))
    z = m.prolong(e)
    y = c.lat.new_field(cs.F32)
    c.op.apply_D(y, z, cs.F32)
    ref = m.restrict(y)
    got = m.coarse_apply(e)
    torch.cuda.synchronize()
    # FP32 sums over an aggregate (768 terms per chirality) on either side: 1e-5
    assert float(torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref)) < 1e-5
