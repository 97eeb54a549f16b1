"""The CFL maximum that a fix-up forms again, when one workgroup takes several
tiles of flagged cells: a blast across the upper and lower z boundary of a box
of 2400 tiles, whose first and last tiles a grid of 1024 (batch, level) or 2048
(single box) workgroups gives to the same ones.  The three forms share the
tiles out in different ways and must find the same dt, to the last bit."""
import numpy as np
import pytest

from paper_2609_10816_amd import ctmhd, inputs

pytestmark = pytest.mark.gpu

SHAPE = (96, 80, 80)
STEPS = 4


def _blast():
    n0, n1, n2 = SHAPE
    x, y, z = ((np.arange(n) + 0.5) / n - 0.5 for n in SHAPE)
    Z, Y, X = np.meshgrid(z, y, x, indexing="ij")
    zd = np.abs(Z + 0.5)
    zd = np.minimum(zd, 1.0 - zd)  # distance from the z boundary
    bf = np.zeros((3, n2, n1, n0))
    bf[0] = bf[1] = 10.0 / np.sqrt(2)
    cons = inputs.from_primitives(np.ones((n2, n1, n0)), np.zeros((3, n2, n1, n0)),
                                  np.where(X ** 2 + Y ** 2 + zd ** 2 < 0.01, 1e3, 0.1), bf)
    return cons, bf, [1.0 / n for n in SHAPE]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_dt_after_fixups(precision):
    cons, bf, dx = _blast()
    P = ctmhd.make_params(recon="ppm", emf="q26", precision=precision)
    cs, bs, dts, ds = ctmhd.run(P, cons, bf, dx, STEPS)
    assert (ds[:, 1] > 0).any() and (ds[:, 3] == 0).all()  # fix-ups of the second stage
    outs, dtb, db = ctmhd.run_batched(P, [(cons, bf, dx)], nsteps=STEPS)
    np.testing.assert_array_equal(dtb[:, 0], dts)
    np.testing.assert_array_equal(db, ds)
    assert np.array_equal(outs[0][0], cs) and np.array_equal(outs[0][1], bs)
    cuts = ((0, 48, 96), (0, 80), (0, 80))
    _, _, dtl, dl = ctmhd.run_level(P, cons, bf, dx, cuts, nsteps=STEPS)
    np.testing.assert_array_equal(dtl, dts)
    np.testing.assert_array_equal(dl[:, :2], ds[:, :2])
