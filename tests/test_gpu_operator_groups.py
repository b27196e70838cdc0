"""The operator's kernels for several right-hand sides at every size of group
and remainder, launched as one workgroup per tile and as a persistent grid:
each right-hand side gets the bits of its own call."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu

NRHS = 7


@pytest.fixture(scope="module")
def case():
    return Case((4, 8, 12, 8), 0.3, 0.1355, 1.0, 101, oracle_T=False, antiperiodic_t=True)


@pytest.mark.parametrize("prec", [cs.F32, cs.F16, cs.BF16])
@pytest.mark.parametrize("tile,workgroups", [(2, 0), (3, 0), (4, 5), (5, 0), (6, 3), (7, 0)])
def test_groups_equal_columns(case, prec, tile, workgroups):
    c = case
    bd = c.to_dev(synth.source(c.dims, 102, nrhs=NRHS), prec)
    one = c.lat.field_bytes(prec)
    out = c.lat.new_field(prec, NRHS)
    c.op.apply_D_cfg(out, bd, prec, NRHS, cs.LaunchConfig(tile, workgroups, 0))
    for r in range(NRHS):
        ref = c.op.apply_D(c.lat.new_field(prec), bd[r * one:(r + 1) * one].clone(), prec)
        assert torch.equal(ref, out[r * one:(r + 1) * one])
