"""Sizes of the meet kernels' work units: the blocks of a launch must end together.

Times are the least of several runs on the device's clock, compared within one
process; the bounds lie between what equal and unequal units take.  Counts are
integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

SEED, ISEED = 21, 9


def _meet_ms(G, q, runs=7):
    return min(S.simrank_single_source_ex(G, q)[2].meet_ms for _ in range(runs))


# Pairs with long tails (c = 0.95, segments of one step) take several rounds of
# units where short ones take one.  The bound lies between one round's time, 1.12
# times that of units of 32 nodes, and several's, 0.96.
def test_long_walks_take_units_of_their_length():
    g = inputs.erdos_renyi_in(20000, 8.0, seed=1)
    G = S.load_csr(g)
    S.simrank_build_index(G, seg_log2=0, kappa=1.0, c=0.95, seed=ISEED)
    q = S.make_query(1, c=0.95, seed=SEED, R=2000, mode=S.MODE_STITCHED)
    auto = _meet_ms(G, q)
    S.simrank_set_tuning(G, 32, 0)
    fixed = _meet_ms(G, q)
    print(f"long walks: {auto:.3f} ms, units of 32 nodes {fixed:.3f}", flush=True)
    assert auto < 1.04 * fixed
    G.free()


# one block's worth of work and several rounds of it, lone and beside a query of
# short walks
@pytest.mark.parametrize("n, R, c, L", [(1, 5, 0.95, 255), (300, 700, 0.99, 255), (20000, 1521, 0.95, 64)])
def test_long_walks_equal_oracle(n, R, c, L):
    g = inputs.erdos_renyi_in(n, 3.0, seed=n)
    G = S.load_csr(g)
    vs = np.unique(np.linspace(0, n - 1, 40).astype(np.int32))
    qs = [S.make_query(0, c=c, seed=SEED, walk_cap=L, R=R), S.make_query(n - 1, seed=SEED, R=R)]
    want = [O.meet_counts_plain(g, 0, SEED, c, L, R, vs), O.meet_counts_plain(g, n - 1, SEED, 0.6, 64, R, vs)]
    assert np.array_equal(S.simrank_single_source_ex(G, qs[0])[1][vs], want[0])
    for cnt, w in zip(S.simrank_batch([G], qs)[1], want):
        assert np.array_equal(cnt[vs], w)
    G.free()


# Two tiles of source walks, the second of so few that its units reach the most
# nodes, and beside it queries of less than a round: in front, behind, both.
@pytest.mark.parametrize("order", [(0, 1), (1, 0), (1, 0, 2), (0, 1, 2)])
def test_small_queries_beside_one_of_unequal_tiles(order):
    gs = [inputs.erdos_renyi_in(60000, 8.0, seed=2), inputs.erdos_renyi_in(700, 5.0, seed=3),
          inputs.erdos_renyi_in(2500, 5.0, seed=4)]
    Gs, Rs = [S.load_csr(g) for g in gs], [7000, 9502, 900]
    qs = [S.make_query(3, seed=SEED + i, R=Rs[i], graph=i) for i in order]
    cnts = S.simrank_batch(Gs, qs)[1]
    for i, cnt in zip(order, cnts):
        vs = np.unique(np.linspace(0, gs[i].n - 1, 60).astype(np.int32))
        assert np.array_equal(cnt[vs], O.meet_counts_plain(gs[i], 3, SEED + i, 0.6, 64, Rs[i], vs)), i
        lone = S.simrank_single_source_ex(Gs[i], S.make_query(3, seed=SEED + i, R=Rs[i]))[1]
        assert np.array_equal(cnt, lone), i
    for G in Gs:
        G.free()


# Large graphs in front of small ones, whose units would start last, and the same
# queries the other way round.  The bound lies between 1.06 where the list's order is
# the launch's and 1 where it is not.
def test_order_of_a_batch_does_not_set_its_time():
    sizes = [150001, 150001, 40000, 5000, 500, 500, 500]
    Gs = {n: S.load_csr(inputs.erdos_renyi_in(n, 8.0, seed=1)) for n in set(sizes)}
    vs = np.arange(40)
    front = [(n, 7 + i, 3 + i) for i, n in enumerate(sizes)]
    ms, counts = [], []
    for order in (front, front[::-1]):
        plan = S.BatchPlan([Gs[n] for n, _, _ in order],
                           [S.make_query(s, seed=k, R=9502, graph=i) for i, (_, s, k) in enumerate(order)])
        best = []
        for _ in range(7):
            plan.run()
            best.append(plan.wait().ms)
        ms.append(min(best))
        counts.append([plan.read(i, want_out=False)[1] for i in range(len(order))])
        plan.free()
    print(f"large graphs in front {ms[0]:.3f} ms, behind {ms[1]:.3f}", flush=True)
    for a, b in zip(counts[0], counts[1][::-1]):
        assert np.array_equal(a, b)
    small = inputs.erdos_renyi_in(500, 8.0, seed=1)
    for i in (4, 5, 6):
        _, s, k = front[i]
        assert np.array_equal(counts[0][i][vs], O.meet_counts_plain(small, s, k, 0.6, 64, 9502, vs))
    assert ms[0] < 1.03 * ms[1]
    for G in Gs.values():
        G.free()


# The tuner keeps units sized on the device where they are fastest: on a small
# graph the best fixed size takes three times as long.
def test_tuner_keeps_units_sized_on_the_device():
    g = inputs.erdos_renyi_in(500, 8.0, seed=1)
    G = S.load_csr(g)
    q = S.make_query(1, seed=SEED, R=2000)
    before, want = _meet_ms(G, q), S.simrank_single_source_ex(G, q)[1]
    t = S.simrank_tune_ex(G, q)
    after = _meet_ms(G, q)
    print(f"tuner: {before:.4f} ms before, {after:.4f} after, {t}", flush=True)
    assert after < 1.75 * before and t["meet_ms"] < 1.75 * before
    assert t["unit_nodes"] in (32, 64, 128, 256)
    assert np.array_equal(S.simrank_single_source_ex(G, q)[1], want)
    S.simrank_set_tuning(G, t["unit_nodes"], 0)          # the fixed size it reports
    assert np.array_equal(S.simrank_single_source_ex(G, q)[1], want)
    G.free()
