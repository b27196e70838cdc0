"""Handles built in memory that earlier handles gave back: same results as the
first ones, for one and several host threads with streams of their own."""
import threading

import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 8)


def _step(lat, U, b, kappa, stream):
    """One operator's life: build, solve (workspace, graphs), force, destroy."""
    with torch.cuda.stream(stream):
        op = cs.Operator(lat, U, kappa, 1.0)
        bd = lat.import_field(b, cs.F64)
        xd = lat.new_field(cs.F64).zero_()
        op.gcr_solve(xd, bd, cs.SolverParams(max_iter=3, tol=0.0), allow_fail=True)
        g, _ = op.force(xd, bd)
        op.bicgstab_solve(xd, bd, cs.SolverParams(max_iter=1, tol=0.0), allow_fail=True)
        out = xd.view(torch.float64).clone(), g.clone()
        stream.synchronize()
        return out


@pytest.mark.parametrize("threads", [1, 3])
def test_rebuilt_handles_give_the_same_results(threads):
    lat = cs.Lattice(DIMS)
    Us = [torch.from_numpy(synth.gauge_field(DIMS, 0.3, 50 + i)).cuda() for i in range(threads)]
    b = torch.from_numpy(synth.source(DIMS, 60)).cuda()
    torch.cuda.synchronize()
    kappas = [0.12 + 0.005 * i for i in range(threads)]
    ref = [_step(lat, Us[i], b, kappas[i], torch.cuda.Stream()) for i in range(threads)]
    bad = []

    def run(i):
        s = torch.cuda.Stream()
        for _ in range(4):
            for x, y in zip(_step(lat, Us[i], b, kappas[i], s), ref[i]):
                if not torch.equal(x, y):
                    bad.append(i)

    ts = [threading.Thread(target=run, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
