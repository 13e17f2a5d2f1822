"""Tensor-parallel degrees that are no powers of two on the 32-bit kernels, which a batch takes by itself
(the 32-bit path cannot be asked for by name there): quotients of the fused rows by multiplication, against
the oracle's divisions."""
import numpy as np
import pytest

import oracle
from paper_2509_24859_amd import workloads as W

from helpers import (assert_plans_equal, oracle_plan_exact_threaded, oracle_plan_h1f1b_threaded, oracle_plan_threaded,
                     simple_problem)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(harp):
    c = harp.Context(0)
    yield c
    c.close()


CASES = [  # L, devices per group, degrees, stage counts, scale of the times
    (2, (3, 2), (1, 2, 3), (2, 2), 1),
    (65, (7, 6, 5), (1, 3, 5, 6, 7), (3, 9), 1),
    (130, (12, 12), (1, 2, 3, 4, 6, 12), (2, 8), 37),
    (300, (13, 11), (1, 11, 13), (2, 20), 1),                    # the second launches: rows beyond a wavefront's share
    (700, (9, 9), (1, 3, 9), (2, 6), 1),
    (48, (6, 6), (1, 2, 3, 6), (2, 6), 1 << 13),                 # sums that leave 32 bits
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "L%d_q%s" % (c[0], "_".join(map(str, c[2]))))
def test_odd_degrees_against_the_oracle(harp, ctx, case):
    L, ndev, degrees, stages, scale = case
    rng = np.random.default_rng(L)
    G = len(ndev)
    bw = rng.integers(20, 60, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 700
    p = simple_problem(np.zeros(L), M=9, T=2, G=G, ndev=ndev, tp=degrees, gtype=[g % 2 for g in range(G)],
                       fwd=rng.integers(1, 900, size=(2, L)) * scale, bwd=rng.integers(1, 900, size=(2, L)) * scale,
                       act=rng.integers(10, 3000, size=L) * scale, params=rng.integers(0, 40, size=L),
                       stash=rng.integers(0, 10, size=L), bw=bw)
    p.type_mem_bytes[:] = 90 * L // sum(ndev) + 100
    tables = harp.Tables(ctx, p)
    assert not tables.fast32
    cands = W.make_candidates(p, L, 77, max(G, stages[0]), max(G, stages[1]), 0, 48 if L < 500 else 12)
    ot = oracle.build_tables(p)
    want = oracle_plan_threaded(ot, cands)
    got, _ = harp.plan(ctx, p, cands)
    assert_plans_equal(got, want, "min-max")
    assert (want.status == oracle.OK).any()
    if L <= 130:
        got, _, _ = harp.plan_exact(ctx, p, cands)
        assert_plans_equal(got, oracle_plan_exact_threaded(ot, cands), "exact")
    else:                                                           # the oracle's sweep takes too long there
        got, n, _ = harp.plan_exact(ctx, p, cands)
        wide, n_wide, _ = harp.plan_exact(ctx, p, cands, harp.PATH_GENERIC)
        assert_plans_equal(got, wide, "exact")
        assert (n == n_wide).all()
    caps = np.where(want.status == oracle.OK, want.bottleneck + want.bottleneck // 8, 7)
    got, _ = harp.plan_h1f1b(ctx, p, cands, caps)
    h = oracle_plan_h1f1b_threaded(ot, cands, caps)
    assert_plans_equal(got, h, "H-1F1B")
    assert (got.warmup == h.warmup).all()


@pytest.mark.parametrize("degree", [3, 6, 7, 641, 65535])
@pytest.mark.parametrize("beyond", [False, True], ids=["last", "beyond"])
def test_quotients_at_the_end_of_their_range(harp, ctx, degree, beyond):
    """Fused rows that end one below 2^31, and one beyond, where the int64 kernels take over."""
    L = 6
    total = (1 << 31) - 1 - (degree - 1) + (1 if beyond else 0)     # row[L] + degree - 1 = 2^31 - 1, or 2^31
    fwd = np.full(L, total // L, dtype=np.int64)
    fwd[-1] += total - fwd.sum()
    p = simple_problem(np.zeros(L), M=3, G=2, ndev=(degree, degree), tp=(1, degree), fwd=fwd[None, :],
                       bwd=np.zeros((1, L), dtype=np.int64), act=[0] * L, bw=[[9, 9], [9, 9]])
    from helpers import cands_from_lists
    cands = cands_from_lists([[(0, degree)], [(0, 1)], [(0, degree), (1, 1)], [(1, 1), (0, degree)], [(0, degree), (1, degree)]])
    want = oracle.plan_batch(oracle.build_tables(p), cands)
    got, _ = harp.plan(ctx, p, cands)
    assert_plans_equal(got, want, "degree %d" % degree)
    got, _, _ = harp.plan_exact(ctx, p, cands)
    assert_plans_equal(got, oracle_plan_exact_threaded(oracle.build_tables(p), cands), "exact, degree %d" % degree)
