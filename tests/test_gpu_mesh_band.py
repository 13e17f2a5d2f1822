"""The band-limited kernels of the submesh planner at the edges of their tiles: 64 columns, 64 cuts per
mask word, four degrees per step, value rows beyond LDS, the orderings they hand over, and the small
problems that are worked as whole tables instead."""
import numpy as np
import pytest

import oracle
from paper_2509_24859_amd import workloads as W

from helpers import (assert_plans_equal, oracle_plan_mesh_h1f1b_sweep_threaded, oracle_plan_mesh_h1f1b_threaded,
                     oracle_plan_mesh_threaded, simple_problem)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(harp):
    c = harp.Context(0)
    yield c
    c.close()


def _problem(seed, L, ndev, tp, slow=False, scale=1, distinct_links=False):
    rng = np.random.default_rng(seed)
    G = len(ndev)
    bw = rng.integers(20, 60, size=(G, G)) * (1 if not slow else 10)
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = np.arange(G) + 500 if distinct_links else 500
    if slow and G > 1:
        bw[0, 1] = bw[1, 0] = 1                 # one link decides the bottleneck: wide rows
    p = simple_problem(np.zeros(L), M=6, T=2, G=G, ndev=ndev, tp=tp, gtype=[g % 2 for g in range(G)],
                       fwd=rng.integers(1, 900, size=(2, L)) * scale, bwd=rng.integers(1, 900, size=(2, L)) * scale,
                       act=rng.integers(100, 3000, size=L) * scale, params=rng.integers(0, 40, size=L),
                       stash=rng.integers(0, 10, size=L), bw=bw)
    p.type_mem_bytes[:] = 60 * L // max(1, len(ndev)) + 100
    return p


CASES = [  # L, devices per group, degrees, stage counts, slow link, scale of the times, distinct own links
    (2, (1, 1), (1,), (2,), False, 1, False),
    (63, (31, 32), (1, 2, 4, 8, 16), (5, 9), False, 1, False),
    (64, (32, 32), (1, 2, 4, 8, 16, 32), (4, 7), True, 1, False),
    (65, (33, 32), (1, 2, 4, 8, 16), (6, 8), True, 1, False),
    (129, (64, 65), (1, 2, 4, 8, 16, 32, 64, 128), (4, 6), False, 1, False),
    (30, (3, 2, 4), (1, 2, 4), (3, 5, 9), True, 1 << 14, False),       # small: whole table, sums beyond 2^31
    (20, (4, 4), (1, 2, 4), (3, 5), False, 1, False),                  # small: whole table
    (59, (10, 12), (1,), (21, 22), False, 1, False),                   # one degree: whole table
    (90, (10, 12, 9), (1, 2, 4), (9, 12), True, 1 << 13, False),        # sums that leave 32 bits times a degree
    (900, (1, 1, 1, 1), (1, 2, 4, 8, 16, 32, 64, 128), (4,), False, 1, True),   # time rows beyond LDS: handed over
    (400, (32, 32), (1, 2, 4, 8, 16, 32), (8,), True, 1, False),       # value rows beyond LDS
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "L%d_D%d_q%d" % (c[0], sum(c[1]), len(c[2])))
def test_band_kernels_at_their_edges(harp, ctx, case):
    L, ndev, tp, stages, slow, scale, distinct = case
    p = _problem(L, L, ndev, tp, slow, scale, distinct)
    assert harp.Tables(ctx, p).fast32
    G = len(ndev)
    lists = [(S, order) for S in stages for order in (list(range(G)), list(range(G))[::-1])]
    orders = W.orderings_from_lists(lists, S_max=max(stages))
    ot = oracle.build_tables(p)
    want = oracle_plan_mesh_threaded(ot, orders)
    assert (want.status == oracle.OK).any()
    fast, _ = harp.plan_mesh(ctx, p, orders, False, harp.PATH_FAST32)
    assert_plans_equal(fast, want, "min-max")
    assert (fast.stage_tp == want.stage_tp).all() and (fast.stage_group == want.stage_group).all()
    # the exact form against the int64 kernel, which shares no search code with it
    exact, _ = harp.plan_mesh(ctx, p, orders, True, harp.PATH_FAST32)
    wide, _ = harp.plan_mesh(ctx, p, orders, True, harp.PATH_GENERIC)
    assert_plans_equal(exact, wide, "exact")
    assert (exact.stage_tp == wide.stage_tp).all() and (exact.n_passes == wide.n_passes).all()
    # H-1F1B counts under caps at and above the bottleneck
    caps = np.where(want.status == oracle.OK, want.bottleneck + np.arange(orders.C) * want.bottleneck // 7, -1)
    hw = oracle_plan_mesh_h1f1b_threaded(ot, orders, caps)
    hg, _ = harp.plan_mesh_h1f1b(ctx, p, orders, caps, harp.PATH_FAST32)
    assert_plans_equal(hg, hw, "h1f1b")
    assert (hg.warmup == hw.warmup).all() and (hg.stage_tp == hw.stage_tp).all()


ROW_FORMS = [  # L, devices per group, degrees, stages, slow link
    (40, (8, 9), (1, 2), 11, False),                      # every row in LDS for good, two lanes of four with a degree
    (96, (24, 24), (1, 2, 4, 8), 9, False),
    (160, (64, 64), (1, 2, 4, 8), 20, True),              # rows that fit as values and not as key rows
    (160, (64, 64), (1, 2, 4, 8, 16), 18, True),          # five degrees: a lane takes all of a cell's
    (250, (64, 64), (1, 2, 4), 36, True),                 # rows of the workspace
]


@pytest.mark.parametrize("case", ROW_FORMS, ids=lambda c: "L%d_D%d_q%d" % (c[0], sum(c[1]), len(c[2])))
@pytest.mark.parametrize("copies", [1, 300], ids=["few", "many"])
def test_band_rows_in_every_form(harp, ctx, case, copies):
    """Rows of a pass all in LDS, the last two there as values or as key rows, or none of them; a whole compute unit's
    LDS for an ordering and half of it."""
    L, ndev, tp, S, slow = case
    p = _problem(L + S, L, ndev, tp, slow)
    orders = W.orderings_from_lists([(s, order) for s in (S, S - 2) for order in ([0, 1], [1, 0])] * copies, S_max=S)
    want = oracle_plan_mesh_threaded(oracle.build_tables(p), W.orderings_from_lists(
        [(s, order) for s in (S, S - 2) for order in ([0, 1], [1, 0])], S_max=S))
    assert (want.status == oracle.OK).any()
    got, _ = harp.plan_mesh(ctx, p, orders, False, harp.PATH_FAST32)
    for field in ("splits", "dev_first", "bottleneck", "iter_time", "status", "stage_group", "stage_tp"):
        assert (getattr(got, field).reshape(copies, 4, -1) == getattr(want, field).reshape(1, 4, -1)).all(), field
    exact, _ = harp.plan_mesh(ctx, p, orders, True, harp.PATH_FAST32)
    wide, _ = harp.plan_mesh(ctx, p, W.orderings_from_lists(
        [(s, order) for s in (S, S - 2) for order in ([0, 1], [1, 0])], S_max=S), True, harp.PATH_GENERIC)
    for field in ("splits", "dev_first", "bottleneck", "iter_time", "status", "stage_group", "stage_tp", "n_passes"):
        assert (getattr(exact, field).reshape(copies, 4, -1) == getattr(wide, field).reshape(1, 4, -1)).all(), field


@pytest.mark.parametrize("L", [134, 136, 137, 142, 144, 145, 160, 162, 163, 169, 171, 172])
def test_layouts_that_just_fit(harp, ctx, L):
    """512 devices in 16 groups of a type each, six degrees: LDS layouts from some room to spare to none at all, in each of the
    band kernels' forms (up to 136 the search over the cap, to 144 the exact form, to 162 H-1F1B's, to 171 min-max), against the int64
    kernels."""
    G, S_max = 16, 24
    rng = np.random.default_rng(L)
    p = simple_problem(np.zeros(L), M=6, T=G, G=G, ndev=[32] * G, tp=(1, 2, 4, 8, 16, 32), gtype=list(range(G)),
                       fwd=rng.integers(1, 30, size=(G, L)), bwd=rng.integers(1, 30, size=(G, L)), act=rng.integers(10, 300, size=L),
                       params=rng.integers(0, 40, size=L), stash=rng.integers(0, 10, size=L), bw=rng.integers(20, 60, size=(G, G)),
                       mem=[200 * L] * G)
    orders = W.orderings_from_lists([(S, order) for S in (17, S_max) for order in (list(range(G)), list(range(G))[::-1])], S_max=S_max)
    assert harp.Tables(ctx, p).fast32
    fields = ("splits", "dev_first", "bottleneck", "iter_time", "status", "stage_group", "stage_tp")
    want, _ = harp.plan_mesh(ctx, p, orders, False, harp.PATH_GENERIC)
    assert (want.status == oracle.OK).any()
    caps = np.where(want.status == oracle.OK, want.bottleneck + np.arange(orders.C) * want.bottleneck // 7, -1)
    for run, more in ((lambda path: harp.plan_mesh(ctx, p, orders, False, path)[0], ()),
                      (lambda path: harp.plan_mesh(ctx, p, orders, True, path)[0], ("n_passes",)),
                      (lambda path: harp.plan_mesh_h1f1b(ctx, p, orders, caps, path)[0], ("warmup",)),
                      (lambda path: harp.plan_mesh_h1f1b_sweep(ctx, p, orders, path=path)[0], ("warmup", "t_max", "n_caps"))):
        fast, wide = run(harp.PATH_FAST32), run(harp.PATH_GENERIC)
        for field in fields + more:
            assert (getattr(fast, field) == getattr(wide, field)).all(), field


FIRST_CAPS = [  # L, devices per group, degrees, stages, slow link: which of them decides, few and many stages
    (30, (14, 14), (1,), 28, False),
    (30, (14, 14), (1,), 28, True),
    (32, (14, 14), (1, 2), 24, True),
    (32, (14, 14), (1, 2), 25, True),
    (90, (8, 9), (1, 2, 4), 9, False),
    (90, (8, 9), (1, 2, 4), 9, True),
]


@pytest.mark.parametrize("case", FIRST_CAPS, ids=lambda c: "L%d_S%d_%s" % (c[0], c[3], "link" if c[4] else "speeds"))
def test_first_caps(harp, ctx, case):
    """Orderings whose first cap is tried at once and ones that search first, against the int64 kernels."""
    L, ndev, tp, S, slow = case
    p = _problem(3 * L + S, L, ndev, tp, slow)
    orders = W.orderings_from_lists([(s, order) for s in (S, S - 1) for order in ([0, 1], [1, 0])] * 80, S_max=S)
    for run, more in ((lambda path: harp.plan_mesh(ctx, p, orders, False, path)[0], ()),
                      (lambda path: harp.plan_mesh(ctx, p, orders, True, path)[0], ("n_passes",)),
                      (lambda path: harp.plan_mesh_h1f1b_sweep(ctx, p, orders.slice(0, 4), path=path)[0], ("warmup", "t_max", "n_caps"))):
        fast, wide = run(harp.PATH_FAST32), run(harp.PATH_GENERIC)
        assert (wide.status == oracle.OK).any()
        for field in ("splits", "dev_first", "bottleneck", "iter_time", "status", "stage_group", "stage_tp") + more:
            assert (getattr(fast, field) == getattr(wide, field)).all(), field


def test_a_first_cap_above_which_there_is_none(harp, ctx):
    """The cheapest cut of the only link takes 2^31 - 1 us: the first cap is the largest there is."""
    L = 90
    p = _problem(7, L, (8, 9), (1, 2, 4))
    p.act_bytes[:] = 2 ** 31 - 1
    p.bw[0, 1] = p.bw[1, 0] = 1
    p.bw[0, 0] = p.bw[1, 1] = 2 ** 31
    assert harp.Tables(ctx, p).fast32
    orders = W.orderings_from_lists([(s, order) for s in (5, 9) for order in ([0, 1], [1, 0])], S_max=9)
    want = oracle_plan_mesh_threaded(oracle.build_tables(p), orders)
    assert (want.status == oracle.OK).all() and (want.bottleneck == 2 ** 31 - 1).all()
    got, _ = harp.plan_mesh(ctx, p, orders, False, harp.PATH_FAST32)
    assert_plans_equal(got, want, "min-max")


RUN_LENGTHS = [  # as above: entries of a reach table that a thread works, between one and eight, and a row's last run cut short
    (255, (5, 4), (1, 2, 4), 4, False),
    (511, (8, 8), (1, 2, 4, 8), 5, True),
    (1000, (8, 9), (1, 2, 4, 8), 4, False),
]


@pytest.mark.parametrize("case", RUN_LENGTHS, ids=lambda c: "L%d_q%d" % (c[0], len(c[2])))
@pytest.mark.parametrize("copies", [1, 80, 300])
def test_reach_tables_by_runs(harp, ctx, case, copies):
    """Workgroups of every size over tables of one to several entries a thread."""
    test_band_rows_in_every_form(harp, ctx, case, copies)


@pytest.mark.parametrize("seed,L,ndev,tp,M", [(1, 33, (3, 4), (1, 2, 4), 9), (2, 64, (4, 4, 2), (1, 2), 5),
                                              (3, 70, (2, 2, 2), (1, 2), 40), (4, 20, (8,), (1, 2, 4, 8), 12)],
                         ids=lambda x: str(x).replace(" ", ""))
def test_band_sweep_equals_the_exhaustive_one(harp, ctx, seed, L, ndev, tp, M):
    """The bounded search over the cap against the kernels that try every cap (int64 path): plans that open
    at the bottleneck, climbs to a larger cap (memory that only fits smaller counts), sweeps cut short."""
    rng = np.random.default_rng(seed)
    G = len(ndev)
    climbs = 0
    for tight in (10, 7, 5, 4):
        bw = rng.integers(2, 40, size=(G, G))
        bw = np.minimum(bw, bw.T)
        bw[np.arange(G), np.arange(G)] = 60
        p = simple_problem(np.zeros(L), M=M, T=2, G=G, ndev=ndev, tp=tp, gtype=[g % 2 for g in range(G)],
                           fwd=rng.integers(1, 300, size=(2, L)), bwd=rng.integers(1, 300, size=(2, L)),
                           act=rng.integers(100, 4000, size=L), params=rng.integers(0, 20, size=L),
                           stash=rng.integers(1, 40, size=L), bw=bw)
        p.type_mem_bytes[:] = tight * L * 10 // sum(ndev)
        orders = W.make_orderings(p, seed, 5, G, min(L, sum(ndev)), 0, 12)
        for max_caps in (1 << 20, 1, 2, 11):
            fast, _ = harp.plan_mesh_h1f1b_sweep(ctx, p, orders, max_caps, harp.PATH_FAST32)
            wide, _ = harp.plan_mesh_h1f1b_sweep(ctx, p, orders, max_caps, harp.PATH_GENERIC)
            assert_plans_equal(fast, wide, "memory %d, at most %d caps" % (tight, max_caps))
            for name in ("stage_group", "stage_tp", "warmup", "t_max", "n_caps"):
                assert (getattr(fast, name) == getattr(wide, name)).all(), (tight, max_caps, name)
        mm, _ = harp.plan_mesh(ctx, p, orders)
        ok = mm.status == oracle.OK
        at, _ = harp.plan_mesh_h1f1b(ctx, p, orders, np.where(ok, mm.bottleneck, -1))
        climbs += int((ok & (at.status != oracle.OK)).sum())
    assert climbs > 0


def _opening_beyond_the_end(seed):
    """Problems whose memory only fits once a large cap has lowered the warm-up counts: such a cap can be
    above t_E = ceil(T / M) of its own plan (it exceeds that plan's sum by M or more)."""
    if seed < 0:
        rng, L = np.random.default_rng(0), 24
        p = simple_problem(np.zeros(L), M=4, G=1, ndev=(4,), tp=(1, 2), fwd=rng.integers(30, 60, size=(1, L)),
                           bwd=np.zeros((1, L), dtype=np.int64), act=np.full(L, 5000), stash=[4] + [0] * (L - 1), mem=[5],
                           bw=[[1000]], ar_count=0)
        return p, W.orderings_from_lists([(2, [0])])
    rng = np.random.default_rng(seed)
    L, ndev = int(rng.integers(5, 14)), ((1, 1), (2, 1), (2, 2), (3,))[seed % 4]
    G, M = len(ndev), int(rng.integers(2, 6))
    bw = rng.integers(2, 5, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 60
    p = simple_problem(np.zeros(L), M=M, T=2, G=G, ndev=ndev, tp=(1, 2) if max(ndev) > 1 else (1,),
                       gtype=[g % 2 for g in range(G)], fwd=rng.integers(1, 6, size=(2, L)),
                       bwd=rng.integers(1, 6, size=(2, L)), params=rng.integers(0, 4, size=L),
                       act=np.where(rng.random(L) < 0.6, rng.integers(0, 7, size=L), rng.integers(300, 900, size=L)),
                       stash=rng.integers(0, 10, size=L), bw=bw)
    p.type_mem_bytes[:] = rng.integers(4, 10) * L // sum(ndev)
    return p, W.make_orderings(p, seed, 5, 2, min(L, sum(ndev)), 0, 4)


def test_band_sweep_opening_beyond_its_own_end(harp, ctx):
    """Every cap up to the first one with a plan counts as tried, also those above the t_E which that plan
    fixes, and max_caps cuts the climb to it: against the oracle."""
    beyond = 0
    for seed in range(-1, 40):
        p, orders = _opening_beyond_the_end(seed)
        ot = oracle.build_tables(p)
        full = oracle_plan_mesh_h1f1b_sweep_threaded(ot, orders)
        limits = {1, 1 << 20}
        for n in full.n_caps[full.status == oracle.OK]:
            limits.update(int(x) for x in range(max(1, n - 4), n + 2))
        for max_caps in sorted(limits):
            want = oracle_plan_mesh_h1f1b_sweep_threaded(ot, orders, max_caps)
            got, _ = harp.plan_mesh_h1f1b_sweep(ctx, p, orders, max_caps, harp.PATH_FAST32)
            assert_plans_equal(got, want, "seed %d, at most %d caps" % (seed, max_caps))
            for name in ("stage_group", "stage_tp", "warmup", "t_max", "n_caps"):
                assert (getattr(got, name) == getattr(want, name)).all(), (seed, max_caps, name)
        # a sweep that opens above its own end has nothing left to try
        beyond += int(((full.status == oracle.OK) & (full.t_max > -(-full.iter_time // p.M))).sum())
    assert beyond >= 5


# (form, L, types, groups, degrees, S_max, devices per group): LDS of the band kernels within 288 bytes of 160 KiB
FULL_LDS = [("min-max", 882, 6, 3, 7, 50, 22), ("exact", 318, 7, 6, 8, 16, 3), ("exact", 528, 8, 8, 4, 32, 8),
            ("h1f1b", 349, 7, 7, 7, 202, 1), ("sweep", 603, 5, 4, 6, 57, 1)]


@pytest.mark.parametrize("form,L,T,G,n_tp,S_max,n", FULL_LDS, ids=lambda x: str(x))
def test_shapes_that_would_fill_the_lds(harp, ctx, form, L, T, G, n_tp, S_max, n):
    """Shapes whose dynamic LDS alone would fit a compute unit, and not together with what the band kernels
    hold statically: they run on the whole-table kernels.  Against the int64 path."""
    rng = np.random.default_rng(L)
    bw = rng.integers(20, 60, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 500
    p = simple_problem(np.zeros(L), M=6, T=T, G=G, ndev=(n,) * G, tp=[1 << k for k in range(n_tp)],
                       gtype=[g % T for g in range(G)], fwd=rng.integers(1, 900, size=(T, L)),
                       bwd=rng.integers(1, 900, size=(T, L)), act=rng.integers(100, 3000, size=L), bw=bw)
    assert harp.Tables(ctx, p).fast32
    S = G if n == 1 else min(G * n, S_max)
    orders = W.orderings_from_lists([(S, list(range(G))), (S, list(range(G))[::-1])], S_max=S_max)
    if form in ("min-max", "exact"):
        got, want = (harp.plan_mesh(ctx, p, orders, form == "exact", path)[0] for path in (harp.PATH_FAST32, harp.PATH_GENERIC))
    elif form == "h1f1b":
        caps = harp.plan_mesh(ctx, p, orders)[0].bottleneck
        got, want = (harp.plan_mesh_h1f1b(ctx, p, orders, caps, path)[0] for path in (harp.PATH_FAST32, harp.PATH_GENERIC))
    else:
        got, want = (harp.plan_mesh_h1f1b_sweep(ctx, p, orders, 9, path)[0] for path in (harp.PATH_FAST32, harp.PATH_GENERIC))
    assert (want.status == oracle.OK).all()
    assert_plans_equal(got, want, form)
    assert (got.stage_tp == want.stage_tp).all() and (got.stage_group == want.stage_group).all()


def _repeated(orders, extra, C):
    """A batch of C orderings: the given ones and the malformed `extra` ones over and over, in a fixed mix."""
    at = np.random.default_rng(C).permutation(np.resize(np.arange(orders.C + len(extra)), C))
    lists = [(int(orders.ord_S[c]), list(orders.ord_group[c, :orders.ord_G[c]])) for c in range(orders.C)] + extra
    many = W.orderings_from_lists([lists[x] for x in at], S_max=orders.S_max, G_max=orders.G_max)
    return at, W.orderings_from_lists(lists, S_max=orders.S_max, G_max=orders.G_max), many


@pytest.mark.parametrize("L,ndev,scale,slow,stages", [
    (75, (40, 34, 2), 1, False, (8, 7, 9, 6)), (75, (40, 34, 2), 1 << 13, False, (8, 7, 9, 6)),
    (140, (40, 34, 2), 1 << 13, True, (64, 60, 63, 26)), (42, (160, 130, 2), 1, False, (22, 21, 19, 12))],
    ids=["in_range", "no_keys", "handed_over", "wide"])
@pytest.mark.parametrize("C", [300, 700, 2500])
def test_band_kernels_on_large_batches(harp, ctx, C, L, ndev, scale, slow, stages):
    """More orderings than compute units (512-thread workgroups), than twice as many (256 threads in the
    min-max form), and than there are workgroups; in range, with sums that leave 32 bits times a degree, and
    with sums that leave 32 bits themselves (the band kernels hand those over).  The batch repeats a few
    orderings, malformed and infeasible ones among them, so the oracle works each once."""
    tp = (1, 2, 4, 8, 16)                               # 77 columns, or 293: more than a workgroup has threads
    p = _problem(7, L, ndev, tp, slow, scale)
    assert harp.Tables(ctx, p).fast32
    orders = W.orderings_from_lists(list(zip(stages, ([0, 1, 2], [2, 1, 0], [1, 0], [0]))), S_max=max(stages) + 3,
                                    G_max=4)
    extra = [(0, [0, 1]), (4, [0, 0]), (5, [0, 3]), (2, [0, 1, 2]), (12, [2])]
    at, few, many = _repeated(orders, extra, C)
    ot = oracle.build_tables(p)
    want = oracle_plan_mesh_threaded(ot, few)
    assert (want.status == oracle.OK).sum() >= 3 and (want.status != oracle.OK).sum() >= 5
    names = ("status", "splits", "dev_first", "bottleneck", "iter_time", "stage_group", "stage_tp")

    def same(got, want, extra_names=()):
        for name in names + extra_names:
            a, b = getattr(got, name), getattr(want, name)[at]
            bad = np.nonzero((a != b).reshape(C, -1).any(axis=1))[0]
            assert bad.size == 0, (name, bad.size, int(at[bad[0]]))

    same(harp.plan_mesh(ctx, p, many, False, harp.PATH_FAST32)[0], want)
    same(harp.plan_mesh(ctx, p, many, True, harp.PATH_FAST32)[0], harp.plan_mesh(ctx, p, few, True, harp.PATH_GENERIC)[0],
         ("n_passes",))
    caps = np.where(want.status == oracle.OK, want.bottleneck // 8 * 9, 0)
    same(harp.plan_mesh_h1f1b(ctx, p, many, caps[at], harp.PATH_FAST32)[0], oracle_plan_mesh_h1f1b_threaded(ot, few, caps),
         ("warmup",))
    limit = 6                                            # caps: the int64 path tries every one
    same(harp.plan_mesh_h1f1b_sweep(ctx, p, many, limit, harp.PATH_FAST32)[0],
         harp.plan_mesh_h1f1b_sweep(ctx, p, few, limit, harp.PATH_GENERIC)[0], ("warmup", "t_max", "n_caps"))


@pytest.mark.parametrize("slow,scale", [(True, 1 << 13), (False, 1), (False, 1 << 13)], ids=["slow_link", "small", "large"])
def test_band_h1f1b_under_loose_caps(harp, ctx, slow, scale):
    """Caps around and beyond 2^31, under which the sums are bounded by the operators instead: the counts
    still follow the cap that was asked for (on the slow link up to 64 times twice 24e6 us, above 2^31)."""
    p = _problem(3, 61, (5, 6), (1, 2, 4), slow, scale)
    assert harp.Tables(ctx, p).fast32
    orders = W.orderings_from_lists([(5, [0, 1]), (7, [1, 0]), (6, [0, 1]), (3, [1])], S_max=8)
    ot = oracle.build_tables(p)
    base = oracle_plan_mesh_threaded(ot, orders)
    assert (base.status == oracle.OK).sum() >= 3
    counts = set()
    top = min((1 << 47) - 1, oracle.INF // (3 * p.L + p.M))
    for cap in (0, (1 << 31) - 2, (1 << 31) - 1, 1 << 31, 3 * 10**9, (1 << 32) + 5, 1 << 40, top, top + 1):
        caps = np.where(base.status == oracle.OK, base.bottleneck, 7) if cap == 0 else np.full(orders.C, cap)
        want = oracle_plan_mesh_h1f1b_threaded(ot, orders, caps)
        got, _ = harp.plan_mesh_h1f1b(ctx, p, orders, caps, harp.PATH_FAST32)
        assert_plans_equal(got, want, "cap %d" % cap)
        assert (got.warmup == want.warmup).all() and (got.stage_tp == want.stage_tp).all(), cap
        counts.add(want.warmup.tobytes())
    assert len(counts) >= 3


def test_band_orderings_without_a_plan(harp, ctx):
    """Tight memory on one of two GPU types, as many stages as devices: the chains, which may leave a stage
    without operators, reach the end on orderings that have no plan, and below the optimum of others."""
    rng = np.random.default_rng(1)
    L, G = 150, 4
    bw = rng.integers(20, 60, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 500
    p = simple_problem(np.zeros(L), M=20, T=2, G=G, ndev=(10,) * G, tp=[1 << k for k in range(8)],
                       gtype=[g % 2 for g in range(G)], fwd=rng.integers(1, 900, size=(2, L)),
                       bwd=rng.integers(1, 900, size=(2, L)), act=rng.integers(100, 3000, size=L),
                       params=rng.integers(0, 40, size=L), stash=rng.integers(1, 20, size=L), bw=bw)
    lists = [(S, [int(g) for g in rng.permutation(G)[:k]]) for S, k in ((40, 4),) * 8 + ((30, 3),) * 6 + ((20, 2),) * 4]
    orders = W.orderings_from_lists(lists, S_max=40)
    some = 0
    for mem in ((1100, 370), (1350, 450), (1500, 400)):
        p.type_mem_bytes[:] = mem
        want = oracle_plan_mesh_threaded(oracle.build_tables(p), orders)
        some += int((want.status != oracle.OK).any() and (want.status == oracle.OK).any())
        for exact in (False, True):
            got, _ = harp.plan_mesh(ctx, p, orders, exact, harp.PATH_FAST32)
            if exact:
                want, _ = harp.plan_mesh(ctx, p, orders, True, harp.PATH_GENERIC)
            assert_plans_equal(got, want, "memory %s, exact %d" % (mem, exact))
            assert (got.stage_tp == want.stage_tp).all() and (got.stage_group == want.stage_group).all()
        got, want = (harp.plan_mesh_h1f1b_sweep(ctx, p, orders, 5, path)[0] for path in (harp.PATH_FAST32, harp.PATH_GENERIC))
        assert_plans_equal(got, want, "memory %s, sweep" % (mem,))
        assert (got.n_caps == want.n_caps).all() and (got.t_max == want.t_max).all()
    assert some >= 2


def _tight_sweep(seed):
    """A random problem of a few groups with memory around what its plans need, orderings of it, a limit of caps."""
    rng = np.random.default_rng(seed)
    G = int(rng.integers(2, 6))
    ndev = tuple(int(x) for x in rng.integers(1, 6, size=G))
    L, M, T = int(rng.integers(max(8, G), 34)), int(rng.choice([2, 3, 5, 8, 20, 62])), int(rng.integers(1, 4))
    bw = rng.integers(20, 900, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 4000
    fwd = np.rint(np.exp(6 + 0.6 * rng.standard_normal((1, L)))).astype(np.int64)
    act = rng.integers(8, 65, size=L) * int(rng.choice([100, 1000, 5000]))
    p = simple_problem(np.zeros(L), M=M, T=T, G=G, ndev=ndev, tp=(1, 2, 4), gtype=[g % T for g in range(G)],
                       fwd=np.concatenate([fwd * (t + 1) for t in range(T)]),
                       bwd=np.concatenate([2 * fwd * (t + 1) for t in range(T)]), act=act, params=2000 * fwd[0],
                       stash=4 * act, bw=bw)
    need = p.param_bytes.sum() + min(M, sum(ndev) / 2) / 2 * p.stash_bytes.sum()
    p.type_mem_bytes[:] = rng.uniform(0.6, 2.5) * rng.uniform(0.6, 1.4, size=T) * need / sum(ndev)
    orders = W.make_orderings(p, seed, 5, G, max(G, min(L, sum(ndev))), 0, int(rng.integers(1, 6)))
    return p, orders, int(rng.choice([1 << 20, 1 << 20, 5, 40, 300]))


def test_band_sweep_left_to_several_workgroups(harp, ctx):
    """Tight memory: orderings whose bounds rule little out leave the rest of their caps to several workgroups,
    and those whose climb fails a few times leave it to the kernels that try every cap, from where it stands.
    Against those kernels from the start (int64 path)."""
    import torch
    shared = climbing = 0
    for seed in range(400):
        p, orders, max_caps = _tight_sweep(seed)
        tables = harp.Tables(ctx, p)
        assert tables.fast32
        do = harp.DeviceOrderings(ctx, orders)
        C, S_max = orders.C, orders.S_max
        out = harp.DevicePlans(ctx, C, S_max)
        ints = [torch.full(n, -7, dtype=torch.int32, device=ctx.device) for n in ((C, S_max), (C, S_max), (C, S_max), (C,))]
        group, tp, warmup, n_caps = ints
        t_max = torch.full((C,), -7, dtype=torch.int64, device=ctx.device)
        ws = harp.mesh_sweep_workspace(ctx, tables, do)
        for _ in range(2):                               # the workspace of one call is lent to the next
            harp.harp_plan_mesh_h1f1b_sweep_batch(ctx, tables, do, max_caps, out, group, tp, warmup, t_max, ws, n_caps)
        want, _ = harp.plan_mesh_h1f1b_sweep(ctx, p, orders, max_caps, harp.PATH_GENERIC)
        assert_plans_equal(out.to_host(), want, "seed %d" % seed)
        for name, got in (("stage_group", group), ("stage_tp", tp), ("warmup", warmup), ("t_max", t_max), ("n_caps", n_caps)):
            assert (got.cpu().numpy() == getattr(want, name)).all(), (seed, name)
        counters = ws[:32].view(torch.int32).tolist()    # of the launch: orderings handed over [1], left to walkers [5]
        climbing, shared = climbing + counters[1], shared + counters[5]
    assert shared >= 3 and climbing >= 3


def test_mesh_workspace_has_a_slice_per_resident_workgroup(harp, ctx):
    """160 operators, 128 devices, 32 stages: two whole-table workgroups of 1,024 threads are resident per
    compute unit, and the band form needs no more slices than those have."""
    import torch
    L, D, S = 160, 128, 32
    p = _problem(1, L, (D // 2, D // 2), (1, 2, 4, 8))
    orders = W.orderings_from_lists([(S, [0, 1])] * 4096)
    do = harp.DeviceOrderings(ctx, orders)
    row = (L + 1) * (D + 1)
    slice_bytes = 24 * row + 4 * S * row                     # two rows of values and counts, back-pointers
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    need = harp.mesh_workspace(ctx, harp.Tables(ctx, p), do).numel()
    assert need <= 2 * n_cu * (slice_bytes + 256) + (1 << 22)     # lists and the feasibility index: below 4 MB
