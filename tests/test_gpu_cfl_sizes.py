"""The CFL step around 4096 cells, up to which one block takes all of them in one
launch: against the formula in numpy (rounding of a dozen operations: 1e-14
relative), and af_step, which saves the state in that launch, against af_run."""
import numpy as np
import pytest
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA, MU, PR, CC, CV = 1.4, 0.01, 0.72, 0.4, 0.1
SIDES = (W.NOSLIP, W.OUTFLOW, W.SYMMETRY, W.NOSLIP)


@pytest.mark.parametrize("n1,n2", [(4, 4), (63, 65), (64, 64), (241, 17), (128, 64), (300, 220)])
def test_dt_and_step(n1, n2):
    g, f = W.random_smooth_2d(n1, n2, seed=n1, bc=SIDES, amp=0.15)
    U = W.make_state(g, f, GAMMA)
    S = af.Solver(g, mu=MU, Pr=PR, cfl_c=CC, cfl_v=CV)
    A, B = S.to_device(U), S.to_device(U)
    r, m1, m2, E = U[:4 * n1 * n2].reshape(4, -1)
    dx, dy = (g.x1 - g.x0) / n1, (g.y1 - g.y0) / n2
    c = np.sqrt(GAMMA * (GAMMA - 1) * (E - 0.5 * (m1 ** 2 + m2 ** 2) / r) / r)
    a = max(((np.abs(m1 / r) + c) / (CC * dx)).max(), ((np.abs(m2 / r) + c) / (CC * dy)).max())
    v = (max(4 * MU / 3, GAMMA * MU / PR) / (CV * min(dx, dy) ** 2) / r).max()
    dt = 1.0 / (a + v)
    assert abs(float(S.af_cfl_dt(A).item()) - dt) <= 1e-14 * dt
    # clipped to t_final
    assert float(S.af_cfl_dt(A, 0.0, 0.25 * dt).item()) == 0.25 * dt
    st, used, h = S.af_step(A)
    assert st == 0 and h == 0 and abs(used - dt) <= 1e-14 * dt
    assert S.af_run(B, 0.0, 1e30, 1, check_every=1)[:2] == (0, 1)
    assert torch.equal(A, B)
