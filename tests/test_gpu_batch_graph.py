"""Batches whose slots are captured in a graph and replayed (more than two slots'
worth of steps), with steps that are redone among them: on strips and on a set
tile variant, against the same slots launched one by one and against single runs,
bit for bit; and runs that t_final alone ends."""
import pytest
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W
from test_gpu_batch import instances, run_single

pytestmark = pytest.mark.gpu
GAMMA = 1.4


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
@pytest.mark.parametrize("tiles", [False, True])
@pytest.mark.parametrize("aps,steps", [(1, 6), (2, 7), (3, 10)])
def test_replayed_slots_with_rejected_attempts(precision, tiles, aps, steps):
    assert steps > 2 * aps  # else nothing is captured
    insts = instances()
    solvers = [af.Solver(g, precision=precision, **kw) for g, f, kw in insts]
    U0 = [S.to_device(W.make_state(g, f, GAMMA)) for S, (g, f, kw) in zip(solvers, insts)]
    B = af.Batch(solvers)
    if tiles:
        B.variant = B.variant
    A, D = [U.clone() for U in U0], [U.clone() for U in U0]
    out = B.af_batch_run(A, 0.0, 1e30, steps, attempts_per_slot=aps, use_graph=True)
    assert out[0] == [af.AF_OK] * len(insts) and out[1] == [steps] * len(insts)
    assert max(out[3]) > steps  # an instance redid a step
    # some eager work, then the slots one by one
    sum(float(a.sum()) for a in A)
    assert B.af_batch_run(D, 0.0, 1e30, steps, attempts_per_slot=aps, use_graph=False) == out
    for (g, f, kw), a, d, t in zip(insts, A, D, out[2]):
        assert torch.equal(a, d)
        ref, tr = run_single(g, f, kw, steps, precision)
        assert t == tr and (a.cpu().numpy() == ref).all()
    # the same batch again, from the same states
    E = [U.clone() for U in U0]
    assert B.af_batch_run(E, 0.0, 1e30, steps, attempts_per_slot=aps, use_graph=True) == out
    assert all(torch.equal(a, e) for a, e in zip(A, E))


@pytest.mark.parametrize("use_graph", [False, True])
def test_the_largest_step_count(use_graph):
    insts = instances()[:2]
    solvers = [af.Solver(g, **kw) for g, f, kw in insts]
    U0 = [S.to_device(W.make_state(g, f, GAMMA)) for S, (g, f, kw) in zip(solvers, insts)]
    B = af.Batch(solvers)
    A, D = [U.clone() for U in U0], [U.clone() for U in U0]
    out = B.af_batch_run(A, 0.0, 2e-4, 10 ** 6, use_graph=use_graph)
    assert B.af_batch_run(D, 0.0, 2e-4, 2 ** 63 - 1, use_graph=use_graph) == out
    assert all(torch.equal(a, d) for a, d in zip(A, D))
    A, D = U0[0].clone(), U0[0].clone()
    one = solvers[0].af_run_graph(A, 0.0, 2e-4, 10 ** 6)
    assert solvers[0].af_run_graph(D, 0.0, 2e-4, 2 ** 63 - 1) == one
    assert torch.equal(A, D)
