"""A plan of the batched or level call holds nothing that its key leaves out:
plans with the same key have the same bytes, so a plan that a call accepts is
one that it would have built itself.  The parameters that a plan does not hold
(eta among them) may change between calls with one plan."""
import itertools

import numpy as np
import pytest

from paper_2609_10816_amd import ctmhd, inputs

BASE = dict(recon="ppm", emf="q26")
CHANGES = [dict(eta=1e-3), dict(eta=2e-3), dict(cfl=0.2), dict(gamma=1.4), dict(riemann="llf"),
           dict(precision="fp32"), dict(precision="fp32_r64"), dict(flag_mask=3),
           dict(fofc=False), dict(recon="plm"), dict(emf="b25a"), dict(emf="fs18"),
           dict(tile=ctmhd.make_tile(chunk=8)), dict(tile=ctmhd.make_tile(strips=2)),
           dict(tile=ctmhd.make_tile(xrows=2)), dict(tile=ctmhd.make_tile(emf_kernel="edge"))]


def _boxes(dx):
    shapes, off, out = [(16, 8, 12), (4, 24, 6), (1, 1, 9)], 0, []
    for n in shapes:
        out.append(ctmhd.make_box(n, 4, dx, off))
        off += int(np.prod([v + 8 for v in n]))
    return out


@pytest.mark.parametrize("level", [False, True])
def test_equal_keys_mean_equal_plans(level):
    plans = []
    for change in [{}] + CHANGES:
        P = ctmhd.make_params(**{**BASE, **change})
        if level:
            boxes = [ctmhd.make_box((8, 6, 5), 4, (0.1,) * 3, k * 16 * 14 * 13) for k in range(2)]
            plan = ctmhd.level_plan(P, boxes, [(0, 0, 0), (8, 0, 0)], (16, 6, 5))
        else:
            plan = ctmhd.batch_plan(P, _boxes((0.1, 0.2, 0.05)))
        plans.append((ctmhd.parse_plan(plan)["key"], plan.tobytes(), change))
    for (k0, b0, c0), (k1, b1, c1) in itertools.combinations(plans, 2):
        assert k0 != k1 or b0 == b1, f"same key, other plan: {c0} and {c1}"


@pytest.mark.parametrize("eta", [1e-3, 0.5])
def test_eta_does_not_change_the_plan(eta):
    boxes = _boxes((0.1, 0.2, 0.05))
    a, b = (ctmhd.batch_plan(ctmhd.make_params(eta=e, **BASE), boxes) for e in (0.0, eta))
    np.testing.assert_array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("level", [False, True])
@pytest.mark.parametrize("built,used", [(0.0, 0.3), (0.3, 0.0), (0.1, 0.4)])
def test_plan_built_for_another_eta(level, built, used):
    """The dt (the resistive limit is a large part of it here) and the state are
    those of a plan built for the call's own eta, to the last bit."""
    import torch
    cons, bf, info = inputs.turbulent_box((16, 12, 8), mach=1.0, seed_v=5, seed_a=6)
    dx = info["dx"]

    def advance(eta_plan):
        P = ctmhd.make_params(eta=eta_plan, **BASE)
        if level:
            cuts = ((0, 8, 16), (0, 12), (0, 8))
            states, origin = ctmhd.split_level(cons, bf, dx, cuts)
            st = ctmhd.BatchedState.from_numpy(states, ctmhd.required_ghosts(P))
            S = ctmhd.LevelStepper(P, st, origin, (16, 12, 8))
        else:
            st = ctmhd.BatchedState.from_numpy([(cons, bf, dx), (cons, bf, [v / 2 for v in dx])],
                                               ctmhd.required_ghosts(P))
            S = ctmhd.BatchedStepper(P, st)
        S.params = ctmhd.make_params(eta=used, **BASE)
        dt = torch.zeros(3, dtype=torch.float64, device="cuda")
        diag = torch.zeros(12, dtype=torch.int64, device="cuda")
        S.step(3, dt_out=dt, diag=diag)
        torch.cuda.synchronize()
        assert (diag.view(3, 4)[:, 3] == 0).all()
        return dt, st.cons + st.bface

    dt, fields = advance(built)
    ref, ref_fields = advance(used)
    assert torch.equal(dt, ref)
    assert all(torch.equal(a, b) for a, b in zip(fields, ref_fields))
