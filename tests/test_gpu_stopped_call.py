"""A call stops at the first step whose dt is not a positive finite number: the
state is that after the steps before it, with its ghost layers, the counters
of the stopped and later steps are [0, 0, 0, 1], and their dt is the bad value,
then 0.  The steps alternate between two buffers (an odd number starts from a
copy), so every parity of the step count and of the stopping step is taken, in
the single-box, batched and level forms."""
import numpy as np
import pytest
import torch

from paper_2609_10816_amd import ctmhd, inputs

pytestmark = pytest.mark.gpu

SHAPE = (19, 12, 9)


def _cold_box():
    """Supersonic random flow: every face pass counts HLL fallbacks."""
    rng = np.random.default_rng(91)
    s = SHAPE[::-1]
    bf = np.ones((3,) + s) * np.array([0.3, 0.2, 0.1]).reshape(3, 1, 1, 1)
    return inputs.from_primitives(0.5 + rng.random(s), 2.0 * rng.normal(size=(3,) + s),
                                  np.full(s, 0.02), bf), bf, [0.1, 0.1, 0.1]


def _advance(form, P, nsteps, dts):
    cons, bf, dx = _cold_box()
    g = ctmhd.required_ghosts(P)
    if form == "box":
        st = ctmhd.BoxState.from_numpy(cons, bf, g, dx)
        S = ctmhd.Stepper(P, st)
    else:
        st = ctmhd.BatchedState.from_numpy([(cons, bf, dx)], g)
        S = ctmhd.BatchedStepper(P, st) if form == "batch" else \
            ctmhd.LevelStepper(P, st, [(0, 0, 0)], SHAPE)
    dt_out = torch.full((max(nsteps, 1),), -1.0, dtype=torch.float64, device="cuda")
    diag = torch.full((4 * max(nsteps, 1),), -1, dtype=torch.int64, device="cuda")
    S.step(nsteps, dt_fixed=torch.tensor(dts, dtype=torch.float64, device="cuda"), dt_out=dt_out,
           diag=diag)
    torch.cuda.synchronize()
    return ([t.flatten().cpu().numpy() for t in st.cons + st.bface], dt_out.cpu().numpy(),
            diag.view(-1, 4).cpu().numpy(), (cons, bf))


@pytest.mark.parametrize("form", ["box", "batch", "level"])
@pytest.mark.parametrize("fofc", [True, False])
@pytest.mark.parametrize("nsteps,bad", [(1, 0), (2, 0), (2, 1), (3, 0), (3, 1), (3, 2), (4, 1),
                                        (4, 2)])
@pytest.mark.parametrize("value", [float("nan"), 0.0])
def test_stopped_call(form, fofc, nsteps, bad, value):
    P = ctmhd.make_params(recon="ppm", emf="q26", fofc=fofc)
    dts = [1e-4 * (k + 1) for k in range(nsteps)]
    ref, rdt, rdiag, start = _advance(form, P, bad, dts[:bad] or [1.0])
    dts[bad] = value
    got, dt, diag, _ = _advance(form, P, nsteps, dts)
    if bad == 0:  # no step ran: the caller's interior values
        g = ctmhd.required_ghosts(P)
        sl = tuple(slice(g, g + n) for n in SHAPE[::-1])
        full = tuple(n + 2 * g for n in SHAPE[::-1])
        got = [t.reshape(full)[sl] for t in got]
        ref = list(start[0]) + list(start[1])
    for a, b in zip(got, ref):
        np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(dt[:bad], rdt[:bad])
    np.testing.assert_array_equal(dt[bad], value)
    assert (dt[bad + 1:] == 0.0).all()
    np.testing.assert_array_equal(diag[:bad], rdiag[:bad])
    assert (diag[bad:] == np.array([0, 0, 0, 1])).all()
    if bad > 0:
        assert diag[0, 2] > 0  # the face passes do count fallbacks here
