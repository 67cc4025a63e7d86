"""1D runs on either side of the size up to which a run's steps fix dt themselves:
blocks of steps against the same steps with dt given by the reduction kernel, and
af_step, bit for bit."""
import pytest
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W
from test_gpu_tiles_1d import field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [53, 1199, 1200, 1201])
@pytest.mark.parametrize("rk", [3, 54])
@pytest.mark.parametrize("bc", [W.PERIODIC, W.OUTFLOW])
def test_blocks_equal_steps_with_given_dt(n, rk, bc):
    g, U, kw = field(n, bc)
    S = af.Solver(g, rk=rk, **kw)
    A, B, D = (S.to_device(U) for _ in range(3))
    t_final = 5.5 * float(S.af_cfl_dt(A).item())
    st, steps, t = S.af_run(A, 0.0, t_final, 6, check_every=3)
    tb = td = 0.0
    for _ in range(steps):
        dt = float(S.af_cfl_dt(B, tb, t_final).item())
        assert S.af_step(B, dt, tb, t_final)[0] == af.AF_OK
        tb += dt
        st, used, h = S.af_step(D, 0.0, td, t_final)
        assert (st, used, h) == (af.AF_OK, dt, 0)
        td += used
    assert steps == 6 and t == tb == td == t_final
    assert torch.equal(A, B) and torch.equal(A, D)
