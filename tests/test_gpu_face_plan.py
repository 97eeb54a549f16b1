"""The face pass of a periodic box solves every face once and stores the
copies that its ghost shell needs; a level (here of one box that covers the
whole domain) solves the shell itself.  The two, and every chunking of the
marches and of the x line, evaluate the same arithmetic on the same values,
so states, dt and counters are the same bit for bit: on boxes of one to a few
cells per axis (many copies), rows that end just below, at and above the 64
cells of a wavefront, and in all reconstructions and edge schemes (shell
widths)."""
import numpy as np
import pytest

from paper_2609_10816_amd import ctmhd, inputs

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (2, 1, 3), (5, 7, 1), (1, 9, 2), (16, 16, 16), (58, 3, 2), (59, 2, 3),
          (60, 4, 1), (64, 5, 4), (61, 33, 8), (130, 6, 17)]


def _state(shape, seed=81):
    """A random state of cold, fast flow: shocks, HLL fallbacks and flagged cells."""
    rng = np.random.default_rng(seed)
    s = shape[::-1]
    u = 3.0 * rng.normal(size=(3,) + s)
    p = 0.02 + 0.5 * rng.random(s)
    A = 0.3 * rng.normal(size=(3,) + s)
    dx = [0.1, 0.12, 0.09]
    bf = 0.1 * inputs.curl_edges(A, dx) + np.array([0.4, 0.2, -0.3]).reshape(3, 1, 1, 1)
    return inputs.from_primitives(0.5 + rng.random(s), u, p, bf), bf, dx


def _run(shape, tile=0, level=False, **kw):
    cons, bf, dx = _state(shape)
    P = ctmhd.make_params(tile=tile, cfl=0.2, **kw)
    if level:
        return ctmhd.run_level(P, cons, bf, dx, [(0, n) for n in shape], 2)
    return ctmhd.run(P, cons, bf, dx, 2)


def _same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("recon,emf,precision", [
    ("pc", "q26", "fp64"), ("plm", "q26", "fp64"), ("ppm", "q26", "fp64"), ("ppm", "b25a", "fp64"),
    ("plm_minmod", "fs18", "fp64"), ("ppm", "q26", "fp32"), ("ppm", "fs18", "fp32_r64")])
def test_copies_equal_solved_shell(shape, recon, emf, precision):
    kw = dict(recon=recon, emf=emf, precision=precision, eta=1e-3)
    one = _run(shape, **kw)
    _same(one, _run(shape, level=True, **kw))
    cons, bf, dx = _state(shape)
    got, dts, diag = ctmhd.run_batched(ctmhd.make_params(cfl=0.2, **kw), [(cons, bf, dx)], 2)
    _same(one, (got[0][0], got[0][1], dts[:, 0], diag))


@pytest.mark.parametrize("shape", SHAPES)
def test_launch_shape_same_bits(shape):
    kw = dict(recon="ppm", emf="q26")
    one = _run(shape, **kw)
    for chunk, xrows in ((1, 1), (3, 2), (7, 5), (64, 64)):
        _same(one, _run(shape, tile=ctmhd.make_tile(chunk=chunk, xrows=xrows), **kw))


def test_bricks_same_bits():
    """A box whose state exceeds the size from which the face pass is cut into
    bricks (ragged, so that edge bricks are partial), against the same box as a
    level of one box, which is not cut."""
    shape = (150, 170, 262)
    cons, bf, info = inputs.turbulent_box(shape, mach=2.0, b0=(0.5, 0.3, -0.2), db_rms=0.2,
                                          seed_v=83, seed_a=84)
    dx = [1.0 / 128.0] * 3
    P = ctmhd.make_params(recon="plm", emf="q26", eta=1e-3)
    _same(ctmhd.run(P, cons, bf, dx, 1),
          ctmhd.run_level(P, cons, bf, dx, [(0, n) for n in shape], 1))
