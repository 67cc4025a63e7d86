"""af_run_graph on one context whose sides change between runs: a periodic axis
has a point less than others, so the states and what lies behind them in the
workspace move, and a graph recorded before reads the wrong places.  Each run
against af_run of a solver made for its sides, bit for bit, there and back."""
import pytest
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

pytestmark = pytest.mark.gpu
P, OUT, NS, SY = W.PERIODIC, W.OUTFLOW, W.NOSLIP, W.SYMMETRY


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
@pytest.mark.parametrize("n1,n2", [(70, 33), (100, 64)])
def test_sides_changed_between_runs(precision, n1, n2):
    sides = [(P, P, P, P), (OUT, OUT, OUT, OUT), (P, P, NS, SY), (P, P, P, P), (NS, OUT, SY, NS)]
    kw = dict(mu=0.01, Pr=0.72, precision=precision)
    grids = [W.random_smooth_2d(n1, n2, seed=3, bc=bc, amp=0.15) for bc in sides]
    # the workspace of the grid with the most points holds that of every other
    S = af.Solver(grids[1][0], **kw)
    for bc, (g, f) in zip(sides, grids):
        R = af.Solver(g, **kw)
        assert R.ws_bytes <= S.ws_bytes
        A = R.to_device(W.make_state(g, f, 1.4))
        B = A.clone()
        for side, kind in enumerate(bc):
            assert af.lib().af_set_bc(S.ctx, side, int(kind)) == af.AF_OK
        for steps in (3, 5):  # recorded, then replayed from the start
            assert S.af_run_graph(B, 0.0, 1e30, steps, attempts_per_slot=2)[:2] == \
                R.af_run(A, 0.0, 1e30, steps)[:2]
            torch.cuda.synchronize()
            assert torch.equal(A, B), (bc, steps)
