"""The rebuilt third row of a link, bit for bit: D without a clover term and
with kappa a power of two takes a spinor with one nonzero entry to its
neighbours as kappa times single link entries, which no later step rounds."""
import numpy as np
import pytest
import torch

from paper_2112_00501_amd import cloversap as cs
from paper_2112_00501_amd import synth

pytestmark = pytest.mark.gpu

DIMS = (8, 8, 8, 8)


def _row2(u):
    """Row 2 of links u[..., 2, 3] in single precision: conj(row 0 x row 1), a complex
    product as a product and an FMA (exact in the wider type, then rounded)."""
    w, f = np.longdouble, np.float32
    re, im = u.real.astype(f), u.imag.astype(f)

    def mul(a, b):  # (ar + i ai)(br + i bi)
        ar, ai, br, bi = a[0].astype(w), a[1].astype(w), b[0].astype(w), b[1].astype(w)
        return (ar * br - (ai * bi).astype(f).astype(w)).astype(f), (ai * br + (ar * bi).astype(f).astype(w)).astype(f)

    def e(r, c):
        return re[..., r, c], im[..., r, c]

    rows = []
    for i, j in ((1, 2), (2, 0), (0, 1)):
        p, q = mul(e(0, i), e(1, j)), mul(e(0, j), e(1, i))
        rows.append((p[0] - q[0]) + 1j * (q[1] - p[1]))
    return np.stack(rows, -1)


def test_third_row_is_rounded_as_stated():
    U = synth.gauge_field(DIMS, 0.3, 121)
    lat = cs.Lattice(DIMS)
    op = cs.Operator(lat, torch.from_numpy(U).cuda(), 0.125, 0.0)
    V = lat.volume
    u = U.reshape(V, 4, 3, 3)
    third = _row2(u[..., :2, :])
    coord = lambda s: [s % 8, s // 8 % 8, s // 64 % 8, s // 512]  # noqa: E731
    site = lambda c: ((c[3] % 8 * 8 + c[2] % 8) * 8 + c[1] % 8) * 8 + c[0] % 8  # noqa: E731
    sites = np.random.default_rng(122).integers(0, V, 16)
    src = np.zeros((3 * len(sites), V, 4, 3), dtype=np.complex128)
    for k, s in enumerate(sites):
        for col in range(3):
            src[3 * k + col, s, 0, col] = 1.0  # spin 0: the upper half of every projector keeps it
    b = lat.import_field(torch.from_numpy(src).cuda(), cs.F32)
    out = lat.export_field(op.apply_D(lat.new_field(cs.F32, len(src)), b, cs.F32, len(src)), cs.F32, len(src))
    out = out.cpu().numpy() * -8
    for k, s in enumerate(sites):
        for mu in range(4):
            c = coord(s)
            c[mu] -= 1
            back = site(c)  # its forward neighbour is s
            for col in range(3):
                assert out[3 * k + col, back, 0, 2] == third[back, mu, col]
