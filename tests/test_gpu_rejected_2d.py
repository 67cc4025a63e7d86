"""The status of a 2D step whose halving is exhausted: that of all flags of the
first flagged stage of the last attempt, as stages launched one by one raise them
(they never stop early), whichever strip or row of the stage meets its flag first;
by af_step, af_run, af_run_graph and a batch, in both precisions.  States with a
NaN, an infinity, a zero or a negative density and a negative energy, which raise
AF_FLAG_NONFINITE beside AF_FLAG_CELL_LOW, and a tube whose steps are too large,
which does not."""
import numpy as np
import pytest
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA = 1.4


def damaged(n1, n2):
    g, f = W.shock_tube_2d(n1, n2)
    U = W.make_state(g, f, GAMMA)
    nc = n1 * n2
    yield "sound", g, U
    for what, at, v in (("nan", nc // 2, np.nan), ("inf", nc + 7, np.inf), ("zero", nc - 3, 0.0),
                        ("negative density", 3, -1.0), ("negative energy", 3 * nc + nc // 3, -1.0),
                        ("nan point", 4 * nc + 5, np.nan), ("nan corner", len(U) - 2, np.nan)):
        V = U.copy()
        V[at] = v
        yield what, g, V


def stage_flags(S, U, dt):
    """flags of the first flagged stage of an RK3 attempt"""
    a, b, c = (torch.empty_like(U) for _ in range(3))
    for k, (src, out) in enumerate(((U, a), (a, b), (b, c))):
        S.af_reset_flags()
        S.af_rk_stage(k, U, src, out, dt=dt)
        fl = S.af_read_flags()
        if fl:
            return fl
    return 0


def status_of(fl):
    return af.AF_E_NONFINITE if fl & 4 else (af.AF_E_PP if fl else af.AF_OK)


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
@pytest.mark.parametrize("limiter", [af.LIM_ALL, af.LIM_PP, af.LIM_SMOOTH | af.LIM_POINT])
@pytest.mark.parametrize("n1,n2", [(24, 12), (130, 90), (260, 517)])
def test_status(precision, limiter, n1, n2):
    seen = set()
    for what, g, U in damaged(n1, n2):
        for halvings in (0, 2):
            print(f"rejected: {n1}x{n2} precision {precision} limiter {limiter} {what}", flush=True)
            kw = dict(mu=1e-3, Pr=0.73, precision=precision, limiter=limiter,
                      max_halvings=halvings)
            S = af.Solver(g, **kw)
            U0 = S.to_device(U)
            sound = S.to_device(next(damaged(n1, n2))[2])
            for dt in (1e-3, 40 * float(S.af_cfl_dt(sound).item())):
                fl = stage_flags(S, U0, dt / 2 ** halvings)
                A = U0.clone()
                st, used, h = S.af_step(A, dt)
                if h > halvings:
                    assert st == status_of(fl) != af.AF_OK
                    assert S.af_read_flags() == fl
                    assert torch.equal(A.view(torch.int64), U0.view(torch.int64))
                    seen.add(st)
                else:
                    assert st == af.AF_OK
            # at the CFL step (0 from a state that gives none, which the loop on
            # the device does not try)
            cfl = float(S.af_cfl_dt(U0).item())
            if cfl > 0.0:
                fl = stage_flags(S, U0, cfl / 2 ** halvings)
                A, B, C = (U0.clone() for _ in range(3))
                one = S.af_run(A, 0.0, 1e30, 1, check_every=1)
                if one[1] == 0:
                    assert one[0] == status_of(fl) != af.AF_OK
                    assert S.af_read_flags() == fl
                    assert S.af_run(A, 0.0, 1e30, 4, check_every=4)[0] == one[0]
                assert S.af_run_graph(B, 0.0, 1e30, 1)[:2] == one[:2]
                batch = af.Batch([S])
                if batch.on_strips:
                    assert batch.af_batch_run([C], 0.0, 1e30, 1)[:2] == ([one[0]], [one[1]])
    assert af.AF_E_NONFINITE in seen
    if limiter == af.LIM_ALL:
        assert af.AF_E_PP in seen
