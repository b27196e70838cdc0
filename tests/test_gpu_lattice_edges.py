"""Clover term and link gradient on lattices at the edges of their kernels'
indexing: one block in a direction (both neighbours of the block are the block
itself), two blocks (both neighbours are the same block), odd block counts,
against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth
from tests.gpu_helpers import Case, rel

pytestmark = pytest.mark.gpu

DIMS = [(4, 4, 4, 4), (4, 8, 12, 4), (12, 4, 4, 8), (8, 20, 4, 12)]


@pytest.mark.parametrize("dims", DIMS)
def test_clover_and_inverse(dims):
    # entries below 2 in size, each a sum of a few hundred products of unit
    # size: 1e-14 as for the other lattices; the inverse multiplies by cond(C) < 10
    c = Case(dims, 0.3, 0.137, 1.3, 31)
    T, Ti = c.op.clover.export(), c.op.clover.export_inverse()
    torch.cuda.synchronize()
    assert np.abs(T.cpu().numpy() - c.T).max() < 1e-14
    assert np.abs(Ti.cpu().numpy() - oracle.clover_inverse_field(dims, c.T)).max() < 1e-13


@pytest.mark.parametrize("antiperiodic", [False, True])
@pytest.mark.parametrize("dims", DIMS)
def test_force(dims, antiperiodic):
    # a few hundred FP64 products per entry, as on the other lattices: 1e-12
    c = Case(dims, 0.3, 0.137, 1.3, 32, oracle_T=False, antiperiodic_t=antiperiodic)
    x, y = synth.source(dims, 33), synth.source(dims, 34)
    g, _ = c.op.force(c.to_dev(x, cs.F64), c.to_dev(y, cs.F64))
    torch.cuda.synchronize()
    gh, gc = oracle.force(dims, c.Uo, c.kappa, c.csw, x, y)
    assert rel(g.cpu().numpy(), gh + gc) < 1e-12
