"""Batches and pipelines at the sizes where the 32-bit candidate kernels change their split of the work."""
import numpy as np
import pytest

import oracle
from paper_2509_24859_amd import workloads as W

from helpers import assert_plans_equal, oracle_plan_threaded, simple_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(harp):
    c = harp.Context(0)
    yield c
    c.close()


def problem(L, G, ndev, degrees, memory, seed):
    rng = np.random.default_rng(seed)
    bw = rng.integers(20, 900, size=(G, G))
    bw = np.minimum(bw, bw.T)
    bw[np.arange(G), np.arange(G)] = 9000
    fwd = rng.integers(1, 60, size=(2, L))
    p = simple_problem(np.zeros(L), M=24, T=2, G=G, ndev=ndev, tp=degrees, gtype=[g % 2 for g in range(G)], fwd=fwd,
                       bwd=2 * fwd, act=rng.integers(1, 60, size=L) * 1000, params=2000 * fwd[0],
                       stash=rng.integers(8, 65, size=L) * 400, bw=bw)
    p.type_mem_bytes[:] = int(memory * (p.param_bytes.sum() + 3 * p.stash_bytes.sum()) / sum(ndev))
    return p


@pytest.mark.parametrize("C", [1, 63, 64, 65, 129, 16383, 16384, 32769, 65600])
def test_a_batch_is_its_candidates(harp, ctx, C):
    """The pre-pass works 64, 128 or 256 candidates per workgroup, whose last may be short; what a candidate gets
    does not depend on the batch it is in."""
    p = problem(11, 3, (4, 3, 5), (1, 2, 4), 2.2, 7)
    cands = W.make_candidates(p, 5, 77, 3, 6, 0, C)
    cands.cand_tp[::17, 0] = 3                     # some malformed ones: both lists fill
    got, _ = harp.plan(ctx, p, cands)
    idx = np.unique(np.r_[0:min(C, 300), max(0, C - 300):C])
    want = oracle_plan_threaded(oracle.build_tables(p), cands.take(idx))
    for field in ("status", "splits", "dev_first", "bottleneck", "iter_time"):
        assert (getattr(got, field)[idx] == getattr(want, field)).all(), field
    mid = np.arange(0, C, max(1, C // 4000))
    alone, _ = harp.plan(ctx, p, cands.take(mid))
    for field in ("status", "splits", "bottleneck", "iter_time"):
        assert (getattr(got, field)[mid] == getattr(alone, field)).all(), field
    if C > 60:
        assert len(np.unique(want.status)) == 3


@pytest.mark.parametrize("S", [2, 3, 64, 65, 66, 128, 129, 200])
def test_pipelines_longer_than_a_wavefront(harp, ctx, S):
    """Back-pointers are followed 64 stages at a time."""
    p = problem(max(12, 2 * S + 7), 2, (130, 120), (1, 2), 400.0, S)
    cands = W.make_candidates(p, S, 77, S, S, 0, 24)
    tables = oracle.build_tables(p)
    got, _ = harp.plan(ctx, p, cands)
    assert_plans_equal(got, oracle_plan_threaded(tables, cands), "min-max")
    assert (got.status == oracle.OK).any()
    exact, passes, _ = harp.plan_exact(ctx, p, cands)
    want, want_passes, _ = harp.plan_exact(ctx, p, cands, harp.PATH_GENERIC)
    assert_plans_equal(exact, want, "exact")
    assert (passes == want_passes).all()


@pytest.mark.parametrize("memory", [1.2, 2.0, 40.0])
@pytest.mark.parametrize("L", [4, 5, 6, 7, 8, 9, 12, 68])
def test_ranges_of_a_few_cuts(harp, ctx, L, memory):
    """Ranges of previous cuts shorter than a window of four, of one and a bit, and empty ones."""
    p = problem(L, 2, (4, 3), (1, 2), memory, L)
    cands = W.make_candidates(p, L, 77, 2, min(4, L), 0, 200)
    got, _ = harp.plan(ctx, p, cands)
    assert_plans_equal(got, oracle_plan_threaded(oracle.build_tables(p), cands), "windows")
