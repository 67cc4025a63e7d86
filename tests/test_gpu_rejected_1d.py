"""1D steps that are rejected, with all stages in one launch: the step size
that a rejected attempt had (fixed inside the step, on grids of several tiles)
is the one that is halved, and the status of an exhausted step is that of the
first stage with a flag, as with a launch per stage, not that of what later
stages make of inadmissible data."""
import numpy as np
import pytest

import oracle as O
from parity import assert_close
from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA = 1.4
B10, B21, B32, B43, B54 = (0.391752226571890, 0.368410593050371, 0.251891774271694,
                           0.544974750228521, 0.226007483236906)
A20, A21, A30, A32, A40, A43, A54 = (0.444370493651235, 0.555629506348765, 0.620101851488403,
                                     0.379898148511597, 0.178079954393132, 0.821920045606868,
                                     0.386708617503269)


def leblanc(n, mu, **kw):
    g, f = W.leblanc_1d(n)
    return g, W.make_state(g, f, GAMMA), dict(mu=mu, Pr=0.75, **kw)


def first_flags(cfg, U, dt, rk):
    """flags of the first flagged stage of an attempt, by the oracle's stages"""
    def fe(V, tau):
        V, fl = O.fe(cfg, V, tau)
        if fl:
            raise StopIteration(fl)
        return V
    try:
        if rk == 3:
            u1 = fe(U, dt)
            fe(0.75 * U + 0.25 * fe(u1, dt), dt)
        else:
            u1 = fe(U, B10 * dt)
            u2 = A20 * U + A21 * fe(u1, B21 / A21 * dt)
            u3 = A30 * U + A32 * fe(u2, B32 / A32 * dt)
            u4 = A40 * U + A43 * fe(u3, B43 / A43 * dt)
            fe(u4, B54 / A54 * dt)
    except StopIteration as s:
        return s.value
    return 0


@pytest.mark.parametrize("n,mu", [(100, 0.0), (200, 1e-5), (800, 1e-5), (4096, 0.0)])
@pytest.mark.parametrize("rk", [3, 54])
@pytest.mark.parametrize("noalloc", [False, True])
def test_a_step_halves_the_dt_it_fixed(n, mu, rk, noalloc):
    g, U, kw = leblanc(n, mu, rk=rk, cfl_c=8.0, cfl_v=2.0)
    cfg = O.make_cfg(g, **kw)
    cfl = O.dt(cfg, U)
    ref = U.copy()
    st, dt, h, _ = O.step(cfg, ref)
    assert st == 0 and h >= 1
    S = af.Solver(g, **kw)
    Ud = S.to_device(U)
    S.af_step(S.to_device(W.make_state(g, lambda x: (1.0 + 0 * x, 0 * x, 1e-6 + 0 * x), GAMMA)))
    stg, dtg, hg = (S.af_step_noalloc if noalloc else S.af_step)(Ud)
    assert (stg, hg) == (af.AF_OK, h)
    assert abs(dtg * 2.0 ** h - cfl) <= 1e-13 * cfl
    # (the bar of a step of the CFL size; the LeBlanc states differ by more orders
    # than a pointwise one could hold)
    assert_close(g, Ud.cpu().numpy(), ref, tol=1e-11, what=f"{n} cells, {h} halvings")


@pytest.mark.parametrize("n,mu,rk,factor", [(100, 0.0, 3, 3), (100, 0.0, 3, 8), (100, 0.0, 3, 12),
                                            (100, 0.0, 54, 5), (100, 0.0, 54, 8),
                                            (100, 0.0, 54, 20), (200, 1e-5, 3, 1),
                                            (200, 1e-5, 3, 10), (200, 1e-5, 54, 1),
                                            (800, 1e-5, 3, 3), (800, 1e-5, 54, 10)])
def test_an_exhausted_step_has_the_first_flags_status(n, mu, rk, factor):
    g, U, kw = leblanc(n, mu, rk=rk)
    cfg = O.make_cfg(g, **kw)
    dt = factor * O.dt(cfg, U)
    fl = first_flags(cfg, U, dt, rk)
    assert fl and not fl & 4
    S = af.Solver(g, max_halvings=0, **kw)
    A = S.to_device(U)
    assert S.af_step(A, dt)[0] == af.AF_E_PP
    # (the first kernel of that stage to raise any)
    assert S.af_read_flags() & ~fl == 0 and S.af_read_flags() != 0
    assert np.array_equal(A.cpu().numpy(), U)
    if factor == 1:
        for every in (1, 8):
            assert S.af_run(A, 0.0, 1e30, 8, check_every=every)[:2] == (af.AF_E_PP, 0)
            assert S.af_read_flags() & ~fl == 0 and S.af_read_flags() != 0
            assert np.array_equal(A.cpu().numpy(), U)
