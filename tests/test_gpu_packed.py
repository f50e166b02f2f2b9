"""Rows packed in 4 bytes (o and degree, a hub's place in a table where the degree
does not fit): queries that gather them must count as those that gather 8 bytes.

Counts are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

ISEED = 9


def _graph(slots, hubs, hub_deg, seed):
    """`slots` edge slots: nodes 2 .. hubs + 1 have hub_deg in-edges (node 2 one
    more, node 3 one less), every fifth of the others none, the rest what is
    left; half of all edges come from hubs and walks meet them all the time."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = max(1000, slots // 8)
    deg = np.zeros(n, np.int64)
    deg[2:hubs + 2] = hub_deg
    if hubs > 1:
        deg[2] += 1
        deg[3] -= 1
    rest = np.arange(hubs + 2, n)
    few = rest[rest % 5 != 0]
    left = slots - int(deg.sum()) - (n - hubs - len(few))   # slots of nodes without in-edges
    deg[few] = left // len(few)
    deg[few[: left - int(deg[few].sum())]] += 1
    assert int(np.maximum(deg, 1).sum()) == slots
    m = int(deg.sum())
    src = np.where(rng.random(m) < 0.5, rng.integers(2, max(hubs, 1) + 2, m), rng.integers(0, n, m))
    off = np.concatenate([[0], np.cumsum(deg)])
    return inputs.CSR(n, off.astype(np.int32), src.astype(np.int32))


def _vs(g):
    return np.unique(np.r_[0:8, np.linspace(8, g.n - 1, 120).astype(int)]).astype(np.int32)


@pytest.fixture(scope="module")
def others():
    """A small graph and one of many hubs, with a query on each and its counts."""
    gs = [inputs.erdos_renyi_in(300, 4.0, seed=1), _graph(2097153, 1400, 1024, 5)]
    Gs = [S.load_csr(g) for g in gs]
    qs = [S.make_query(5, seed=8, R=400, walk_cap=40, graph=1), S.make_query(4, seed=8, R=9000, graph=2)]
    vs = [_vs(g) for g in gs]
    yield Gs, qs, vs, [O.meet_counts_plain(gs[0], 5, 8, 0.6, 40, 400, vs[0]),
                       O.meet_counts_plain(gs[1], 4, 8, 0.6, 64, 9000, vs[1])]
    for G in Gs:
        G.free()


# degrees around the one that just does not fit (2^(32 - b) - 1 for slots of b
# bits); E at the size up to which it is gathered itself, and one slot more; as
# many hubs as the stitched, the plain and the small-tile kernels have rows for,
# and one more (there R is such that small tiles are several)
@pytest.mark.parametrize("slots, hubs, hub_deg", [
    (4000, 0, 0), (524288, 3, 8191), (524289, 3, 4095), (700001, 255, 2000), (1048577, 5, 2047),
    (2097153, 3, 1023), (2097153, 704, 1024), (2097153, 705, 1024), (2097153, 1216, 1024),
    (2097153, 1217, 1024), (4194305, 6848, 512), (4194305, 6849, 512)])
def test_packed_rows_equal_oracle(slots, hubs, hub_deg, others):
    print(f"packed: {slots} slots, {hubs} nodes of in-degree {hub_deg}", flush=True)
    g = _graph(slots, hubs, hub_deg, slots + hubs)
    vs, G = _vs(g), S.load_csr(g)
    R = 9000 if hubs > 700 else 400
    S.simrank_build_index(G, seg_log2=1, kappa=0.05, c=0.6, seed=ISEED)
    qs = [S.make_query(2, seed=3, R=R), S.make_query(g.n - 1, seed=4, R=R, walk_cap=40),
          S.make_query(3, seed=3, R=R, mode=S.MODE_STITCHED)]
    want = [O.meet_counts_plain(g, 2, 3, 0.6, 64, R, vs), O.meet_counts_plain(g, g.n - 1, 4, 0.6, 40, R, vs),
            O.meet_counts_stitched(g, 3, 3, ISEED, 0.6, 64, 2, O.pool_sizes(g, 0.05), R, vs)]
    for q, w in zip(qs, want):                    # lone
        assert np.array_equal(S.simrank_single_source_ex(G, q)[1][vs], w)
    # in one launch with a small graph's query, with a many-hub graph's, with both
    Gs, oq, ovs, owant = others
    for k in ([0], [1], [0, 1]):
        cnts = S.simrank_batch([G] + Gs, qs + [oq[i] for i in k])[1]
        for c, w in zip(cnts, want):
            assert np.array_equal(c[vs], w), k
        for i, c in zip(k, cnts[3:]):
            assert np.array_equal(c[ovs[i]], owant[i]), k
    srv = S.Server(G, max_slots=3, max_R=R, max_L=64)
    ts = [srv.submit(q) for q in qs]
    for t, w in zip(ts, want):
        assert np.array_equal(srv.wait(t)[1][vs], w)
    srv.destroy()
    G.free()


# E and packed rows, with as many hubs as the stratified kernel has rows for and
# one more
@pytest.mark.parametrize("slots, hubs, hub_deg", [
    (524288, 3, 8191), (524289, 3, 4095), (2097153, 1472, 1024), (2097153, 1473, 1024)])
def test_packed_rows_stratified_equal_oracle(slots, hubs, hub_deg, others):
    print(f"packed, stratified: {slots} slots, {hubs} nodes of in-degree {hub_deg}", flush=True)
    g = _graph(slots, hubs, hub_deg, slots + hubs)
    vs, G = _vs(g), S.load_csr(g)
    q = S.make_stratified_query(2, eps=0.1, seed=6)
    want = O.strat_sums(g, 2, 6, O.strat_params(g.n, 0.6, 0.1), vs)
    assert np.array_equal(S.simrank_single_source_stratified(G, q)[2][vs], want)
    Gs, _, ovs, _ = others
    for k in (0, 1):   # in one launch with a small graph's query, with a many-hub graph's
        other = S.make_stratified_query(5, eps=0.2, seed=8, graph=1)
        plan = S.BatchPlan([G, Gs[k]], [q, other], groups=False)
        plan.run()
        plan.wait()
        assert np.array_equal(plan.read_stratified(0)[2][vs], want)
        got = plan.read_stratified(1)[2]
        plan.free()
        assert np.array_equal(got, S.simrank_single_source_stratified(Gs[k], S.make_stratified_query(5, eps=0.2, seed=8))[2])
    srv = S.Server(G, max_slots=4, max_R=4000, max_L=64)   # (room for the sums of n nodes)
    assert np.array_equal(srv.wait_stratified(srv.submit(q))[2][vs], want)
    srv.destroy()
    G.free()


# groups of both kernel shapes and all walks, with as many hubs as they have rows
# for (256 the stratified one of more than 8) and one more; the marks of a
# block's positions (5 and 9 members: part of a word, a second piece)
@pytest.mark.parametrize("members", [5, 9])
@pytest.mark.parametrize("slots, hubs, hub_deg", [
    (524289, 3, 4095), (2097153, 256, 1024), (2097153, 257, 1024), (2097153, 1536, 1024), (2097153, 1537, 1024)])
def test_packed_rows_groups_equal_oracle(slots, hubs, hub_deg, members, others):
    print(f"packed, {members} members: {slots} slots, {hubs} nodes of in-degree {hub_deg}", flush=True)
    g = _graph(slots, hubs, hub_deg, slots + hubs)
    vs, G, small = _vs(g), S.load_csr(g), others[0][0]
    S.simrank_build_index(G, seg_log2=1, kappa=0.05, c=0.6, seed=ISEED)
    src, R = [2 + i for i in range(members)], 300
    plan = S.BatchPlan([G, small], [S.make_query(s, seed=3, R=R) for s in src] +
                       [S.make_query(s, seed=3, R=R, mode=S.MODE_STITCHED) for s in src] +
                       [S.make_stratified_query(s, eps=0.2, seed=6) for s in src] +
                       [S.make_query(s, seed=8, R=R, graph=1) for s in src[:2]])   # a group that reads E
    assert plan.n_groups == 4
    plan.run()
    plan.wait()
    P, Q = O.strat_params(g.n, 0.6, 0.2), O.pool_sizes(g, 0.05)
    for i in (0, members - 1):
        s = src[i]
        assert np.array_equal(plan.read(i)[1][vs], O.meet_counts_plain(g, s, 3, 0.6, 64, R, vs))
        assert np.array_equal(plan.read(members + i)[1][vs],
                              O.meet_counts_stitched(g, s, 3, ISEED, 0.6, 64, 2, Q, R, vs))
        assert np.array_equal(plan.read_stratified(2 * members + i)[2][vs], O.strat_sums(g, s, 6, P, vs))
    lone = S.simrank_single_source_ex(small, S.make_query(src[1], seed=8, R=R))[1]
    assert np.array_equal(plan.read(3 * members + 1)[1], lone)
    plan.free()
    G.free()


def test_all_hubs_and_no_edges():
    """Every node a hub, and a graph of no edges."""
    n = 3000
    rng = np.random.Generator(np.random.PCG64(1))
    off = np.arange(n + 1, dtype=np.int64) * 1400      # 4.2e6 slots: 23 bits, 3000 hubs
    g = inputs.CSR(n, off.astype(np.int32), rng.integers(0, n, n * 1400).astype(np.int32))
    vs, G = _vs(g), S.load_csr(g)
    cnt = S.simrank_single_source_ex(G, S.make_query(7, seed=3, R=300, walk_cap=40))[1]
    assert np.array_equal(cnt[vs], O.meet_counts_plain(g, 7, 3, 0.6, 40, 300, vs))
    G.free()
    e = S.simrank_load_graph(5, np.zeros(6, np.int32), np.zeros(0, np.int32))
    assert S.simrank_single_source_ex(e, S.make_query(1, R=10))[1].tolist() == [0, 10, 0, 0, 0]
    e.free()
