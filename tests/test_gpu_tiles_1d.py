"""1D stages at the edges of the stage kernel's tiles (61 cells and the points
at their lower sides): one cell short, full, one over, a last tile that holds
one point alone, and several tiles, for every kind of side, against the
oracle at the FP64 bar; and runs whose stages fix dt themselves (up to 4096
cells) beside the same steps with dt given by the reduction kernel."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import assert_close, REL_TOL_FP64
from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA = 1.4


def field(n, bc):
    g = W.Grid(dim=1, n1=n, bc=(bc, bc, bc, bc))

    def f(x):
        return (1.0 + 0.3 * np.sin(2 * np.pi * x), 0.5 + 0.4 * np.cos(2 * np.pi * x),
                1.0 + 0.3 * np.sin(4 * np.pi * x + 0.4))
    kw = dict(mu=1e-3, Pr=0.72)
    if bc == W.DIRICHLET:
        kw["bcstate"] = [[1.0, 0.9, 3.0], [1.0, 0.9, 3.0]]
    return g, W.make_state(g, f, GAMMA), kw


@pytest.mark.parametrize("n", [4, 60, 61, 62, 122, 183, 200])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.OUTFLOW, W.NOSLIP, W.SYMMETRY, W.DIRICHLET])
@pytest.mark.parametrize("rk", [3, 54])
def test_step(n, bc, rk):
    g, U, kw = field(n, bc)
    cfg = O.make_cfg(g, gamma=GAMMA, rk=rk, **kw)
    S = af.Solver(g, gamma=GAMMA, rk=rk, **kw)
    Ud = S.to_device(U)
    for _ in range(2):
        st, dt, h, _ = O.step(cfg, U)
        stg, dtg, hg = S.af_step(Ud)
        assert (stg, hg) == (st, h) and abs(dtg - dt) <= 1e-13 * dt
    assert_close(g, Ud.cpu().numpy(), U, tol=REL_TOL_FP64, what=f"{n} cells, side {bc}")


@pytest.mark.parametrize("n", [150, 4096, 4097])
@pytest.mark.parametrize("rk", [3, 54])
def test_run_equals_steps_with_given_dt(n, rk):
    """af_run against af_cfl_dt and af_step with that dt, bit for bit, the
    last step clipped to t_final (blocks of two steps, so that the last block
    ends there: a block's steps beyond t_final combine the state with dt 0,
    which rounds)"""
    g, U, kw = field(n, W.OUTFLOW)
    S = af.Solver(g, gamma=GAMMA, rk=rk, **kw)
    A, B = S.to_device(U), S.to_device(U)
    t_final = 3.5 * float(S.af_cfl_dt(A).item())
    st, steps, t = S.af_run(A, 0.0, t_final, 4, check_every=2)
    tb = 0.0
    for _ in range(steps):
        dt = float(S.af_cfl_dt(B, tb, t_final).item())
        assert S.af_step(B, dt, tb, t_final)[0] == af.AF_OK
        tb += dt
    assert st == af.AF_OK and steps == 4 and t == tb == t_final
    assert torch.equal(A, B)


@pytest.mark.parametrize("n", [4, 45, 46, 52, 53, 54, 90, 107, 300])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.OUTFLOW, W.NOSLIP, W.SYMMETRY, W.DIRICHLET])
def test_step_equals_its_stages(n, bc):
    """the step in one launch against its stages in a launch each, bit for bit,
    at the edges of the step's tiles (53 cells of their own, 45 in SSP-RK54)"""
    g, U, kw = field(n, bc)
    S = af.Solver(g, gamma=GAMMA, **kw)
    A = S.to_device(U)
    dt = float(S.af_cfl_dt(A).item())
    one, two, out = (torch.empty_like(A) for _ in range(3))
    S.af_rk_stage(0, A, A, one, dt=dt)
    S.af_rk_stage(1, A, one, two, dt=dt)
    S.af_rk_stage(2, A, two, out, dt=dt)
    B = A.clone()
    assert S.af_step(B, dt=dt)[0] == 0
    assert torch.equal(B, out)
    # SSP-RK54: with sources of zero, its stages have a launch each as well
    S = af.Solver(g, gamma=GAMMA, rk=54, **kw)
    B, C = A.clone(), A.clone()
    assert S.af_step(B, dt=dt)[0] == 0
    S.af_step_source(C, dt, [torch.zeros_like(A)] * 5)
    assert torch.equal(B, C)


@pytest.mark.parametrize("n", [150, 4097])
@pytest.mark.parametrize("rk", [3, 54])
@pytest.mark.parametrize("check_every", [2, 3, 5])
def test_run_in_blocks_equals_run_in_single_steps(n, rk, check_every):
    """blocks of even and odd numbers of steps, whose time moves between two
    scalars on the device, against steps whose dt the reduction gives: the same
    states and times"""
    g, U, kw = field(n, W.OUTFLOW)
    S = af.Solver(g, gamma=GAMMA, rk=rk, **kw)
    A, B = S.to_device(U), S.to_device(U)
    one = S.af_run(A, 0.5, 1e30, 8, check_every=1)
    assert one[:2] == (0, 8)
    assert S.af_run(B, 0.5, 1e30, 8, check_every=check_every) == one
    assert torch.equal(A, B)
