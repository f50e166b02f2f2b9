"""A group's blocks hold 16-bit marks (the low half of a position's o()): a walk meets where
the whole position is the same, and tiles cut by walks and by positions count
every pair once.

Counts and weighted sums are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

ISEED = 9


def _check(g, R, L, c, sources):
    """Lone, grouped, stitched, stratified and served queries on g, all nodes."""
    G = S.load_csr(g)
    S.simrank_build_index(G, seg_log2=1, kappa=0.02, c=c, seed=ISEED)
    Q, P = O.pool_sizes(g, 0.02), O.strat_params(g.n, c, 0.1, 600, 20)
    want = [O.meet_counts_plain(g, s, 3, c, L, R) for s in sources]
    tails = [O.meet_counts_stitched(g, s, 3, ISEED, c, min(L, 64), 2, Q, R) for s in sources]
    sums = [O.strat_sums(g, s, 3, P) for s in sources]
    plain = [S.make_query(s, c=c, seed=3, R=R, walk_cap=L) for s in sources]
    stitched = [S.make_query(s, c=c, seed=3, R=R, walk_cap=min(L, 64), mode=S.MODE_STITCHED) for s in sources]
    strat = [S.make_stratified_query(s, c=c, eps=0.1, seed=3, z=600, phi=20) for s in sources]
    for i in range(len(sources)):
        assert np.array_equal(S.simrank_single_source_ex(G, plain[i])[1], want[i])
        assert np.array_equal(S.simrank_single_source_ex(G, stitched[i])[1], tails[i])
        assert np.array_equal(S.simrank_single_source_stratified(G, strat[i])[2], sums[i])
    plan = S.BatchPlan([G], plain + stitched + strat)
    assert plan.n_groups == 3
    plan.run()
    plan.wait()
    k = len(sources)
    for i in range(k):
        assert np.array_equal(plan.read(i)[1], want[i])
        assert np.array_equal(plan.read(k + i)[1], tails[i])
        assert np.array_equal(plan.read_stratified(2 * k + i)[2], sums[i])
    plan.free()
    srv = S.Server(G, max_slots=4, max_R=R, max_L=L)
    for q, w in zip(plain + stitched, want + tails):
        assert np.array_equal(srv.wait(srv.submit(q))[1], w)
    srv.destroy()
    G.free()


# nodes whose o() all have the same low half; two marks; a graph whose o() have
# 16 bits, and one slot more
@pytest.mark.parametrize("degs", [[65536] * 24, [32768] * 48, [4096] * 16, [4096] * 15 + [4097]])
def test_equal_marks_are_not_meets(degs):
    print(f"marks: {len(degs)} nodes, {sum(degs)} slots", flush=True)
    n = len(degs)
    rng = np.random.Generator(np.random.PCG64(n))
    off = np.concatenate([[0], np.cumsum(degs)])
    g = inputs.CSR(n, off.astype(np.int32), rng.integers(0, n, int(off[-1])).astype(np.int32))
    _check(g, 700, 64, 0.6, [0, 3, n - 1])


# tiles cut by walks (entries: about 77% of R at c = 0.6) and by positions (19
# a walk at c = 0.9, 39 at 0.95), a second one of a few walks and several
@pytest.mark.parametrize("R, L, c", [(10600, 64, 0.6), (10700, 64, 0.6), (25000, 40, 0.6),
                                     (2500, 255, 0.9), (4000, 255, 0.95)])
def test_tiles_cut_by_walks_and_positions(R, L, c):
    print(f"tiles: R={R} L={L} c={c}", flush=True)
    g = inputs.erdos_renyi_in(60, 3.0, seed=R)
    s = [int(v) for v in np.flatnonzero(g.in_degree() > 0)[:2]]
    _check(g, R, L, c, s)
