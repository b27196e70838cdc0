"""The autotuner times a bounded number of launch shapes, however large the
batch: each tile as a grid and as a persistent launch, four tiles for the
operator and for the FP64 smoother, and below FP64 eight tiles of the smoother
with one lane per site, where a batch of this size cannot be faster with two."""
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from tests.gpu_helpers import Case

pytestmark = pytest.mark.gpu

NRHS = 96


@pytest.mark.parametrize("prec", [cs.F64, cs.F32, cs.F16])
def test_shapes_timed_are_bounded(prec):
    c = Case((8, 8, 16, 32), 0.3, 0.1355, 1.0, 141, oracle_T=False)  # 64 blocks a colour: past 512 visits
    cs.profile_enable()
    try:
        cs.profile_reset()
        sap, d = c.op.autotune(prec, NRHS)
        torch.cuda.synchronize()
        n_sap, n_d = cs.profile_query("sap_halfsweep")[0], cs.profile_query("dslash")[0]
    finally:
        cs.profile_enable(False)
        cs.profile_reset()
    # a shape is run once and timed three times; a smoother run is four half-sweeps
    assert 0 < n_sap <= (8 if prec == cs.F64 else 16) * 4 * 4 and n_sap % 32 == 0
    assert 0 < n_d <= 8 * 4 and n_d % 8 == 0
    assert 1 <= sap.rhs_tile <= NRHS and 1 <= d.rhs_tile <= NRHS
