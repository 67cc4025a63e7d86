"""1D steps that are rejected, with all stages in one launch: the step size
that a rejected attempt had (fixed inside the step, on grids of several tiles)
is the one that is halved."""
import pytest

import oracle as O
from parity import assert_close
from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA = 1.4


def leblanc(n, mu, **kw):
    g, f = W.leblanc_1d(n)
    return g, W.make_state(g, f, GAMMA), dict(mu=mu, Pr=0.75, **kw)


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
