"""Launch shapes the library chooses for batches when the caller names none:
every right-hand side gets the bits of its own call (operator, FP64 residual)
or of the one-right-hand-side-per-workgroup launch (smoother), at batch sizes
on both sides of the lines where the shape changes."""
import numpy as np
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    # 128 blocks, 64 per colour: four right-hand sides are 512 operator
    # workgroups and 256 visits of a colour
    return Case((8, 8, 16, 32), 0.3, 0.1355, 1.0, 81, oracle_T=False, antiperiodic_t=True)


@pytest.mark.parametrize("nrhs", [4, 5, 9, 16])
@pytest.mark.parametrize("prec", [cs.F64, cs.F32, cs.F16, cs.BF16])
def test_operator_batch_equals_columns(case, prec, nrhs):
    c = case
    bd = c.to_dev(synth.source(c.dims, 82, nrhs=nrhs), prec)
    one = c.lat.field_bytes(prec)
    for f in (c.op.apply_D, c.op.apply_Ddag):
        out = f(c.lat.new_field(prec, nrhs), bd, prec, nrhs)
        for r in range(nrhs):
            assert torch.equal(f(c.lat.new_field(prec), bd[r * one:(r + 1) * one].clone(), prec),
                               out[r * one:(r + 1) * one])


@pytest.mark.parametrize("nrhs", [4, 5, 9, 16])
@pytest.mark.parametrize("prec,block", [(cs.F64, "mr"), (cs.F32, "mr"), (cs.BF16, "mr"), (cs.F16, "jacobi"),
                                        (cs.F32, "eo")])
def test_smoother_batch_equals_untiled(case, prec, block, nrhs):
    c = case
    bd = c.to_dev(synth.source(c.dims, 83, nrhs=nrhs), prec)
    x0 = c.to_dev(0.1 * synth.source(c.dims, 84, nrhs=nrhs), prec)
    lanes = 2 if 64 * nrhs <= 256 else 1
    untiled = cs.LaunchConfig(1, 0, lanes)
    for zero in (True, False):
        a, b = x0.clone(), x0.clone()
        if block == "mr":
            c.op.sap_smooth(a, bd, prec, 1, 3, zero, nrhs)
            c.op.sap_smooth_cfg(b, bd, prec, nrhs, untiled, 1, 3, zero)
        else:
            f = c.op.sap_smooth_jacobi if block == "jacobi" else c.op.sap_smooth_eo
            f(a, bd, prec, 1, 3, zero, nrhs)
            f(b, bd, prec, 1, 3, zero, nrhs, untiled)
        assert torch.equal(a, b)


def test_batched_true_residual_equals_single(case):
    c = case
    nrhs = 6  # 768 workgroups: the FP64 residual b - D x runs in tiles
    bs = synth.source(c.dims, 85, nrhs=nrhs)
    p = dict(inner_prec=cs.F64, basis_prec=cs.F64, n_cy=0, restart=2, max_iter=5, tol=1e-12)
    xd = c.lat.new_field(cs.F64, nrhs).zero_()
    c.op.gcr_solve(xd, c.to_dev(bs, cs.F64), cs.SolverParams(rhs_tile=2, **p), nrhs=nrhs, allow_fail=True)
    x = c.to_host(xd, cs.F64, nrhs)
    for r in (0, 5):
        x1 = c.lat.new_field(cs.F64).zero_()
        c.op.gcr_solve(x1, c.to_dev(bs[r], cs.F64), cs.SolverParams(**p), allow_fail=True)
        assert np.array_equal(c.to_host(x1, cs.F64), x[r])
