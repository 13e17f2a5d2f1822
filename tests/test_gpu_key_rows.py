"""The 32-bit rows that the build writes, and the min-max planner on both sides of the line between key rows and value rows: the largest time of any plan
against 2^31 over the largest degree, with degrees of both kinds, rows of one chunk and of several."""
import numpy as np
import pytest

import oracle
from paper_2509_24859_amd import workloads as W

from helpers import assert_plans_equal, cands_from_lists, oracle_plan_exact_threaded, simple_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(harp):
    c = harp.Context(0)
    yield c
    c.close()


def _worst_time(p):
    """The whole sequence on the slowest group, or the largest output over the slowest link."""
    t = oracle.build_tables(p)
    n_tp = len(p.tp_degrees)
    stage = max(int(t.PF[p.group_type[g]][p.L]) + int(t.PR[g][k][p.L]) for g in range(p.G) for k in range(n_tp))
    return max(stage, -(-int(p.act_bytes.max()) // int(p.bw.min())))


@pytest.mark.parametrize("beyond", [-(1 << 20), -1, 0, 5])
@pytest.mark.parametrize("L,degrees,ndev", [(9, (1,), (4, 3)), (70, (1, 2, 4, 8), (8, 9, 8)), (70, (1, 2, 3, 6), (8, 9, 8)),
                                            (300, (1, 5, 7), (9, 8)), (300, (1, 2, 4), (9, 8))],
                         ids=lambda x: str(x).replace(" ", ""))
def test_times_around_the_limit_of_key_rows(harp, ctx, L, degrees, ndev, beyond):
    rng = np.random.default_rng(L + len(degrees))
    G = len(ndev)
    bw = rng.integers(20, 60, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 700
    fwd = rng.integers(1, 2000, size=(1, L))
    p = simple_problem(np.zeros(L), M=9, T=1, G=G, ndev=ndev, tp=degrees, gtype=[0] * G, fwd=fwd,
                       bwd=rng.integers(1, 2000, size=(1, L)), act=rng.integers(10, 30000, size=L),
                       params=rng.integers(0, 40, size=L), stash=rng.integers(0, 10, size=L), bw=bw)
    p.type_mem_bytes[:] = 90 * L // sum(ndev) + 100
    limit = (2 ** 31 - 1) // max(degrees)
    # most of the time in three operators: stages that hold none of them compare small keys with large ones
    rest = limit + beyond - _worst_time(p)
    for i, part in ((0, rest // 2), (L // 2, rest // 3), (L - 1, rest - rest // 2 - rest // 3)):
        p.fwd_us[0, i] += part
    assert _worst_time(p) == limit + beyond
    cands = W.make_candidates(p, L, 5, G, min(L, G * 4), 0, 96)
    ot = oracle.build_tables(p)
    want = oracle.plan_batch(ot, cands)
    assert (want.status == oracle.OK).sum() >= 8
    got, _ = harp.plan(ctx, p, cands)
    assert_plans_equal(got, want, "plans")
    exact, _, _ = harp.plan_exact(ctx, p, cands)                     # (works on those results)
    few = cands.slice(0, cands.C if L < 100 else 6)                  # (the oracle tries every cap)
    best = oracle_plan_exact_threaded(oracle.build_tables(p), few)
    for name in ("status", "splits", "dev_first", "bottleneck", "iter_time"):
        assert (getattr(exact, name)[:few.C] == getattr(best, name)).all(), name


@pytest.mark.parametrize("L", [255, 256, 1023, 1024, 1025])
def test_rows_at_the_edges_of_a_thread(harp, ctx, L):
    """Four entries of a row per thread, 256 apart: stages that end at and around them."""
    rng = np.random.default_rng(L)
    p = simple_problem(np.zeros(L), M=4, T=2, G=2, ndev=(4, 3), tp=(1, 2, 4), gtype=[0, 1], fwd=rng.integers(1, 90, size=(2, L)),
                       bwd=rng.integers(1, 90, size=(2, L)), act=rng.integers(10, 3000, size=L),
                       params=np.ones(L, dtype=np.int64), stash=np.ones(L, dtype=np.int64), bw=np.full((2, 2), 40))
    p.type_mem_bytes[:] = 6 * L
    cands = W.make_candidates(p, L, 3, 2, 5, 0, 12)
    want = oracle.plan_batch(oracle.build_tables(p), cands)
    assert (want.status == oracle.OK).any() and harp.Tables(ctx, p).fast32
    got, _ = harp.plan(ctx, p, cands, harp.PATH_FAST32)
    assert_plans_equal(got, want, "L %d" % L)


def _totals_problem(L, work, all_reduce, idle_type=0):
    """Two groups of one type; `work`: its compute time, `all_reduce`: the degree-2 total; `idle_type`: of a type no group has."""
    rng = np.random.default_rng(L)
    fwd = rng.integers(1, 90, size=(2, L))
    act = np.full(L, 40 * (all_reduce // (4 * L)))                        # 4 act / bw per operator at degree 2
    act[L - 1] += 40 * (all_reduce // 4 - all_reduce // (4 * L) * L)
    fwd[0, L // 2] += work - fwd[0].sum()
    fwd[1, 0] += idle_type
    return simple_problem(np.zeros(L), M=4, T=2, G=2, ndev=(4, 3), tp=(1, 2), gtype=[0, 0], fwd=fwd, bwd=np.zeros_like(fwd),
                          act=act, params=np.ones(L, dtype=np.int64), stash=np.ones(L, dtype=np.int64),
                          bw=np.full((2, 2), 40))


TOTALS = {  # compute time, all-reduce time at degree 2, an idle type's time, 32-bit rows
    "work": (2 ** 31, 4000, 0, False),
    "all-reduce": (9000000, 2 ** 30, 0, False),
    "sum_at_the_limit": (2 ** 30, 2 ** 29, 0, False),                      # and the rounding of the division: 2^31 + 1
    "sum_below": (2 ** 30 - 2, 2 ** 29, 0, True),                          # 2^31 - 1
    "idle_type": (9000000, 4000, 2 ** 31, True),
}


@pytest.mark.parametrize("L", [70, 1024, 1025, 4000])
@pytest.mark.parametrize("why", list(TOTALS) + ["malformed"])
def test_rows_are_written_where_they_are_read(harp, ctx, why, L):
    """Sums on both sides of 2^31, in one part or in their sum: the 32-bit rows are left alone where one part alone says
    that no kernel reads them."""
    work, all_reduce, idle, fast = TOTALS.get(why, (9000000, 4000, 0, False))
    p = _totals_problem(L, work, all_reduce, idle)
    if why == "malformed":
        p.stash_bytes[L - 1] = -1
    tables = harp.Tables(ctx, p, finalize=False)
    rows = p.G * p.n_tp + p.G * p.G
    area = tables.buf[-rows * ((L + 1 + 15) // 16 * 64):]                  # (the rows are the last of the buffer)
    area.fill_(0x5A)
    tables.rebuild()
    if why == "malformed":
        with pytest.raises(harp.HarpError):
            tables.finalize()
    else:
        tables.finalize()
        assert tables.fast32 == fast
    if why != "sum_at_the_limit":
        assert bool((area == 0x5A).all()) == (not fast)
    if fast:
        cands = W.make_candidates(p, L, 3, 2, 5, 0, 12)
        want = oracle.plan_batch(oracle.build_tables(p), cands)
        assert (want.status == oracle.OK).any()
        got, _ = harp.plan(ctx, p, cands, harp.PATH_FAST32)
        assert_plans_equal(got, want, why)


def test_a_row_of_transfers_too_long_for_it_is_not_written(harp, ctx):
    L = 1025
    p = _totals_problem(L, 9000000, 4000)
    p.act_bytes[5] = 2 ** 31
    p.bw[0, 1] = p.bw[1, 0] = 1                                            # 2^31 us; the groups' own links, 2^31 / 40
    tables = harp.Tables(ctx, p, finalize=False)
    pitch = (L + 1 + 15) // 16 * 64
    cuts = tables.buf[-4 * pitch:].view(4, pitch)
    cuts.fill_(0x5A)
    tables.rebuild()
    tables.finalize()
    assert not tables.fast32
    assert [bool((row == 0x5A).all()) for row in cuts] == [False, True, True, False]


def test_as_many_rows_as_there_can_be(harp, ctx):
    """255 groups with two degrees: 65,535 rows of the 32-bit tables."""
    G, L = 255, 300
    rng = np.random.default_rng(5)
    p = simple_problem(np.zeros(L), M=4, T=3, G=G, ndev=[2] * G, tp=(1, 2), gtype=[g % 3 for g in range(G)],
                       fwd=rng.integers(1, 90, size=(3, L)), bwd=rng.integers(1, 90, size=(3, L)), act=rng.integers(10, 3000, size=L),
                       params=np.ones(L, dtype=np.int64), stash=np.ones(L, dtype=np.int64), bw=rng.integers(20, 60, size=(G, G)))
    cands = cands_from_lists([[(int(g), int(t)) for g, t in zip(rng.permutation(G)[:9], rng.integers(1, 3, 9))] for _ in range(24)]
                             + [[(254, 2), (253, 1), (0, 2)], [(0, 1), (254, 1)]])
    want = oracle.plan_batch(oracle.build_tables(p), cands)
    assert (want.status == oracle.OK).all() and harp.Tables(ctx, p).fast32
    got, _ = harp.plan(ctx, p, cands, harp.PATH_FAST32)
    assert_plans_equal(got, want, "255 groups")
