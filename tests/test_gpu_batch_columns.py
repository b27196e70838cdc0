"""A right-hand side's smoother result does not depend on what it is batched
with: every column of a batch has the bits of its own call, on a lattice small
enough for lane pairs, with batches below and above one visit of a colour per
compute unit, and on one past the line between the kernels."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu


# 64 blocks a colour, of which four right-hand sides are 256 visits; 280 blocks a colour
@pytest.mark.parametrize("dims,nrhs", [((8, 8, 16, 32), 4), ((8, 8, 16, 32), 5), ((8, 8, 16, 32), 9),
                                       ((8, 8, 40, 56), 3)])
@pytest.mark.parametrize("prec,block", [(cs.F64, "mr"), (cs.F32, "mr"), (cs.BF16, "mr"), (cs.F16, "mr"),
                                        (cs.F32, "jacobi"), (cs.F16, "jacobi"), (cs.BF16, "eo")])
def test_smoother_columns_equal_own_calls(dims, nrhs, prec, block):
    c = Case(dims, 0.3, 0.1355, 1.0, 111, oracle_T=False, antiperiodic_t=True)
    bd = c.to_dev(synth.source(c.dims, 112, nrhs=nrhs), prec)
    x0 = c.to_dev(0.1 * synth.source(c.dims, 113, nrhs=nrhs), prec)
    f = {"mr": c.op.sap_smooth, "jacobi": c.op.sap_smooth_jacobi, "eo": c.op.sap_smooth_eo}[block]
    one = c.lat.field_bytes(prec)
    for zero in (True, False):
        x = x0.clone()
        f(x, bd, prec, 2, 3, zero, nrhs)
        for r in (0, nrhs // 2, nrhs - 1):
            col = slice(r * one, (r + 1) * one)
            x1 = x0[col].clone()
            f(x1, bd[col].clone(), prec, 2, 3, zero, 1)
            assert torch.equal(x1, x[col])
