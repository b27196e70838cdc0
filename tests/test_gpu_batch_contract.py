"""What a batched solve promises of its columns at the size where the
autotuner and the lone solve differ in lanes per site (at most 256 blocks a
colour, more than 512 visits in all): with rhs_tile given, the bits of the
lone solve, in one batch and in groups; with rhs_tile 0, the tolerance."""
import numpy as np
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu

NRHS = 9  # 64 blocks a colour: 576 visits


@pytest.fixture(scope="module")
def solved():
    c = Case((8, 8, 16, 32), 0.3, 0.1355, 1.0, 131, oracle_T=False)
    bs = synth.source(c.dims, 132, nrhs=NRHS)
    lone = {}
    for r in (0, 4, 8):
        x = c.lat.new_field(cs.F64).zero_()
        st, s = c.op.gcr_solve(x, c.to_dev(bs[r], cs.F64), cs.SolverParams())
        assert st == 0
        lone[r] = c.to_host(x, cs.F64), s[0]["iters"]
    return c, bs, lone


@pytest.mark.parametrize("tile,groups", [(1, 1), (4, 1), (9, 1), (2, 2)])
def test_given_tile_keeps_the_bits(solved, tile, groups):
    c, bs, lone = solved
    xd = c.lat.new_field(cs.F64, NRHS).zero_()
    st, stats = c.op.gcr_solve(xd, c.to_dev(bs, cs.F64), cs.SolverParams(rhs_tile=tile, rhs_groups=groups), nrhs=NRHS)
    x = c.to_host(xd, cs.F64, NRHS)
    assert st == 0
    for r, (x1, iters) in lone.items():
        assert stats[r]["iters"] == iters and np.array_equal(x1, x[r]), r


@pytest.mark.parametrize("groups", [1, 2])
def test_autotuned_tile_keeps_the_tolerance(solved, groups):
    c, bs, lone = solved
    bd = c.to_dev(bs, cs.F64)
    xd = c.lat.new_field(cs.F64, NRHS).zero_()
    st, stats = c.op.gcr_solve(xd, bd, cs.SolverParams(rhs_groups=groups), nrhs=NRHS)
    x = c.to_host(xd, cs.F64, NRHS)
    assert st == 0 and all(s["true_relres"] <= 1e-10 for s in stats)
    res = c.to_host(c.op.apply_D(c.lat.new_field(cs.F64, NRHS), xd, cs.F64, NRHS), cs.F64, NRHS) - bs
    for r in range(NRHS):
        assert np.linalg.norm(res[r]) <= 1.001e-10 * np.linalg.norm(bs[r])
    for r, (x1, _) in lone.items():  # both residuals are at most 1e-10 |b|
        d = c.op.apply_D(c.lat.new_field(cs.F64), c.to_dev(x[r] - x1, cs.F64), cs.F64)
        assert np.linalg.norm(c.to_host(d, cs.F64)) <= 2.01e-10 * np.linalg.norm(bs[r])
