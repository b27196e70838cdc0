"""FP64 right-hand sides in tiles, which the library chooses on lattices whose
links, clover term and a field leave the last-level cache (about 200 thousand
sites on): the operator, and the residual b - D x of the batched solver, whose
columns get the bits of their own calls, an odd remainder included."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 28, 28)  # 200,704 sites, 784 blocks
NRHS = 5


@pytest.fixture(scope="module")
def case():
    lat = cs.Lattice(DIMS, antiperiodic_t=True)
    op = cs.Operator(lat, torch.from_numpy(synth.gauge_field(DIMS, 0.3, 161)).cuda(), 0.13, 1.0)
    b = lat.new_field(cs.F64, NRHS)
    b.view(torch.float64).normal_(generator=torch.Generator(device="cuda").manual_seed(162))
    torch.cuda.synchronize()
    return lat, op, b


def _kernels(f):
    """Names of the operator's kernels that f() launches."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        f()
        torch.cuda.synchronize()
    return {e.key for e in p.key_averages() if "k_dslash" in e.key}


def test_operator_columns(case):
    lat, op, b = case
    one = lat.field_bytes(cs.F64)
    for f in (op.apply_D, op.apply_Ddag):
        out = lat.new_field(cs.F64, NRHS)
        ran = _kernels(lambda: f(out, b, cs.F64, NRHS))
        assert ran and all("k_dslash_tiled" in k for k in ran), ran
        for r in range(NRHS):
            ref = f(lat.new_field(cs.F64), b[r * one:(r + 1) * one].clone(), cs.F64)
            assert torch.equal(ref, out[r * one:(r + 1) * one]), r


def test_residual_columns(case):
    lat, op, b = case
    one = lat.field_bytes(cs.F64)
    # no smoother, three iterations in cycles of two: first residual, restart, last residual
    p = dict(inner_prec=cs.F64, basis_prec=cs.F64, n_cy=0, restart=2, max_iter=3, tol=1e-12, use_graph=False)
    x = b.clone().view(torch.float64).mul_(0.1).view(torch.uint8).contiguous()
    x0 = x.clone()
    stats = []
    ran = _kernels(lambda: stats.extend(op.gcr_solve(x, b, cs.SolverParams(rhs_tile=1, **p), NRHS, allow_fail=True)[1]))
    assert any("k_dslash_tiled" in k for k in ran), ran
    for r in range(NRHS):
        col = slice(r * one, (r + 1) * one)
        x1 = x0[col].clone()
        _, s1 = op.gcr_solve(x1, b[col].clone(), cs.SolverParams(**p), allow_fail=True)
        assert s1[0]["iters"] == stats[r]["iters"] == 3 and s1[0]["true_relres"] == stats[r]["true_relres"], r
        assert torch.equal(x1, x[col]), r
