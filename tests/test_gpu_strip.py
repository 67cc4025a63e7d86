"""The strip kernel of the 2D stage at the edges of its split: grids one
column short of, at and past a strip's 60 columns, as small as a grid may be,
one row short of and past a range of rows, with every pairing of side kinds.
Against the oracle at the FP64 bar (FP32 stencils: the mixed bar of its own
tests, 1e-5), and bit for bit against the tile kernel, which a batch runs once
a variant is set; with the dt reduction inside the device-resident loop, and
in batches, as well."""
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
SIDES = [(P, P, P, P), (OUT, OUT, OUT, OUT), (NS, NS, NS, SY), (SY, OUT, NS, SY), (P, P, NS, SY),
         (OUT, NS, P, P), (NS, OUT, SY, NS)]
SIZES = [(4, 4), (5, 9), (59, 13), (60, 17), (61, 40), (62, 70), (119, 33), (121, 64)]


def tile_batch(S):
    B = af.Batch([S])
    B.variant = B.variant  # the tiles of its default variant, not strips
    return B


def field(n1, n2, bc):
    g, f = W.random_smooth_2d(n1, n2, seed=n1 + n2, bc=bc, amp=0.15)
    return g, W.make_state(g, f, GAMMA), dict(mu=0.01, Pr=0.72)


@pytest.mark.parametrize("n1,n2", SIZES)
@pytest.mark.parametrize("bc", SIDES)
def test_step_matches_the_oracle_and_the_tile_kernel(n1, n2, bc):
    g, U, kw = field(n1, n2, bc)
    cfg = O.make_cfg(g, gamma=GAMMA, **kw)
    ref = U.copy()
    st, dt, h, _ = O.step(cfg, ref)
    for precision in (af.PREC_FP64, af.PREC_MIXED):
        print(f"strip: {n1}x{n2} sides {bc} precision {precision}", flush=True)
        S = af.Solver(g, precision=precision, **kw)
        A, B, C = (S.to_device(U) for _ in range(3))
        assert S.af_run(A, 0.0, 1e30, 1, check_every=1)[:2] == (st, 1)
        tol = REL_TOL_FP64 if precision == af.PREC_FP64 else 1e-5
        assert_close(g, A.cpu().numpy(), ref, tol=tol, what=f"{n1}x{n2} {bc} prec {precision}")
        assert tile_batch(S).af_batch_run([B], 0.0, 1e30, 1)[1] == [1]
        assert torch.equal(A, B)
        # two steps of the device loop: the second one's dt comes from the stage
        S.af_run_graph(C, 0.0, 1e30, 2)
        S.af_run(A, 0.0, 1e30, 1, check_every=1)
        assert torch.equal(A, C)


@pytest.mark.parametrize("n2", [499, 500, 511])
def test_long_columns_match_the_tile_kernel(n2):
    """row ranges of several lengths, and more strips than compute units"""
    g, U, kw = field(1100, n2, (NS, OUT, SY, NS))
    S = af.Solver(g, **kw)
    A, B = S.to_device(U), S.to_device(U)
    S.af_run(A, 0.0, 1e30, 1, check_every=1)
    tile_batch(S).af_batch_run([B], 0.0, 1e30, 1)
    assert torch.equal(A, B)


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
@pytest.mark.parametrize("sizes", [[(130, 70)], SIZES[6:], SIZES * 9, [(8, 200)] * 40],
                         ids=["one", "two", "many", "narrow"])
@pytest.mark.parametrize("use_graph", [False, True])
def test_batches_match_tiles_and_single_runs(precision, sizes, use_graph):
    """instances of one strip and of many, launched together, over several
    steps: each opens its next step from the maxima its own last stage left;
    and narrow grids, which a batch runs on tiles"""
    Ss, Us = [], []
    for i, (n1, n2) in enumerate(sizes):
        g, U, kw = field(n1, n2, SIDES[i % len(SIDES)])
        Ss.append(af.Solver(g, precision=precision, **kw))
        Us.append(Ss[-1].to_device(U))
    A, T, R = ([U.clone() for U in Us] for _ in range(3))
    B = af.Batch(Ss)
    out = B.af_batch_run(A, 0.0, 1e30, 5, attempts_per_slot=2, use_graph=use_graph)
    B.variant = B.variant
    assert B.af_batch_run(T, 0.0, 1e30, 5, attempts_per_slot=2, use_graph=use_graph) == out
    for S, a, t, r in zip(Ss, A, T, R):
        S.af_run(r, 0.0, 1e30, 5)
        assert torch.equal(a, t) and torch.equal(a, r)
