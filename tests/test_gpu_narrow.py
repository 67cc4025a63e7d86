"""Single grids of few columns and many rows, which run on tiles: on either side
of the rule's line in both precisions (fifteen columns are the most that it
takes), one step of either integrator and one stage under a given blend against
the oracle at the FP64 bar (FP32 stencils: the mixed bar of its own tests, 1e-5),
and a run with the decisions on the device against one with the host's, bit for
bit, with a step that is redone among them."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import assert_close, REL_TOL_FP64
from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
GAMMA = 1.4
P, OUT, NS, SY = W.PERIODIC, W.OUTFLOW, W.NOSLIP, W.SYMMETRY
# either side of the line: FP64 about 2100 rows, FP32 stencils about 4700
SIZES = [(15, 1800), (15, 2500), (4, 4200), (9, 5200), (16, 5200)]


def field(n1, n2, bc):
    g, f = W.random_smooth_2d(n1, n2, seed=n1 + n2, bc=bc, amp=0.15)
    return g, W.make_state(g, f, GAMMA), dict(mu=0.01, Pr=0.72)


@pytest.mark.parametrize("n1,n2", SIZES)
@pytest.mark.parametrize("bc", [(P, P, P, P), (NS, OUT, SY, NS)])
def test_steps_and_runs(n1, n2, bc):
    g, U, kw = field(n1, n2, bc)
    for rk in (3, 54):
        ref = U.copy()
        assert O.step(O.make_cfg(g, gamma=GAMMA, rk=rk, **kw), ref)[0] == 0
        for precision in (af.PREC_FP64, af.PREC_MIXED):
            print(f"narrow: {n1}x{n2} sides {bc} rk {rk} precision {precision}", flush=True)
            S = af.Solver(g, precision=precision, rk=rk, **kw)
            A, B = S.to_device(U), S.to_device(U)
            assert S.af_step(A)[0] == af.AF_OK
            tol = REL_TOL_FP64 if precision == af.PREC_FP64 else 1e-5
            assert_close(g, A.cpu().numpy(), ref, tol=tol, what=f"{n1}x{n2} {bc} rk {rk}")
            if rk == 3:
                R, T = B.clone(), B.clone()
                one = S.af_run(R, 0.0, 1e30, 3)
                assert S.af_run_graph(B, 0.0, 1e30, 3, attempts_per_slot=2)[:3] == one
                assert torch.equal(B, R)
                af.Batch([S]).af_batch_run([T], 0.0, 1e30, 3)
                assert torch.equal(T, R)


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
def test_a_rejected_step(precision):
    """near vacuum and steps too large: attempts are redone with half the step"""
    g, f = W.double_rarefaction(12, 5200, speed=2.0, angle=1.5707963267948966)
    S = af.Solver(g, mu=1e-3, Pr=0.72, cfl_c=4.0, cfl_v=1.0, precision=precision)
    A, B = (S.to_device(W.make_state(g, f, GAMMA)) for _ in range(2))
    one = S.af_run(A, 0.0, 1e30, 4, check_every=1)
    out = S.af_run_graph(B, 0.0, 1e30, 4, attempts_per_slot=3)
    assert out[:3] == one and out[3] > out[1]
    assert torch.equal(A, B)


@pytest.mark.parametrize("n1,n2", SIZES)
def test_a_given_blend(n1, n2):
    g, U, kw = field(n1, n2, (NS, OUT, SY, NS))
    cfg = O.make_cfg(g, gamma=GAMMA, **kw)
    dt = O.dt(cfg, U)
    theta = np.random.default_rng(n1).uniform(0, 1, O.nfaces(cfg)).astype(np.float32)
    ref, fl = O.fe_blend(cfg, U, dt, theta.astype(np.float64))
    assert fl == 0
    for precision in (af.PREC_FP64, af.PREC_MIXED):
        S = af.Solver(g, precision=precision, **kw)
        A = S.to_device(U)
        out, used = torch.empty_like(A), torch.empty(S.face_count, device="cuda")
        S.af_rk_stage_blend(0, A, A, out, dt=dt, theta=torch.from_numpy(theta).cuda(),
                            theta_s_out=used)
        tol = REL_TOL_FP64 if precision == af.PREC_FP64 else 1e-5
        assert_close(g, out.cpu().numpy(), ref, tol=tol, what=f"{n1}x{n2} blend")
        assert np.array_equal(used.cpu().numpy(), theta)
