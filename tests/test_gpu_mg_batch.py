"""The adaptive multigrid setup solves the coarse systems of all null vectors
side by side; its result must be that of M_MG applied to one null vector after
another.  Counts below, at and past the group of right-hand sides that shares
a matrix load, for the fused (nc = 16, 32, 64) and the general product."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 16)


@pytest.fixture(scope="module")
def case():
    return Case(DIMS, 0.3, 0.1355, 1.0, 71, oracle_T=False)


def _blocks(f, nv):
    """nv F32 fields as complex128 [nv][aggregate][chirality][1536 entries]."""
    nblk = DIMS[0] * DIMS[1] * DIMS[2] * DIMS[3] // 256
    t = f.view(torch.float32).view(nv, nblk, 2, 3, 256, 2, 2)  # rows 0..2 upper, 3..5 lower chirality
    return torch.view_as_complex(t.double().contiguous()).reshape(nv, nblk, 2, -1)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("nv", [1, 3, 5, 8, 16, 20, 32])
def test_adaptive_pass_is_the_preconditioner_on_each_vector(case, nv, half):
    c = case
    etas = c.lat.new_field(cs.F32, nv)
    etas.view(torch.float32).normal_(generator=torch.Generator(device="cuda").manual_seed(72))
    kw = dict(nv=nv, coarse_prec=cs.F16 if half else cs.F32)
    v = c.lat.new_field(cs.F32, nv)
    c.op.sap_smooth(v, etas, cs.F32, n_cy=4, n_mr=4, nrhs=nv)
    mg0 = cs.Multigrid(c.op, etas, cs.MgParams(n_adapt=0, **kw))
    one = c.lat.field_bytes(cs.F32)
    z = torch.cat([mg0.apply(v[i * one:(i + 1) * one]) for i in range(nv)])
    P, _ = cs.Multigrid(c.op, etas, cs.MgParams(n_adapt=1, **kw)).export()
    torch.cuda.synchronize()
    # Gram-Schmidt in double precision on every aggregate and chirality
    q = _blocks(z, nv)
    for i in range(nv):
        for j in range(i):
            q[i] -= (q[j].conj() * q[i]).sum(-1, keepdim=True) * q[j]
        q[i] /= torch.linalg.vector_norm(q[i], dim=-1, keepdim=True)
    # single precision through the smoother, the coarse solve and Gram-Schmidt
    # (whose vectors lose up to a factor of ten of their norm): 1e-5
    assert float(torch.linalg.vector_norm(_blocks(P, nv) - q) / torch.linalg.vector_norm(q)) < 1e-5
