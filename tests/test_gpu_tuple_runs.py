"""Algorithm 2's tuple form by runs of start nodes: tuples of one (j, step), or
of several steps, sorted and linked in LDS.  Counts and weighted sums must equal
the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu


def _graph(n_active):
    """n_active nodes with in-edges (two each where they differ), 40 without."""
    n = n_active + 40
    rng = np.random.Generator(np.random.PCG64(n_active))
    dst = np.sort(rng.choice(n, size=n_active, replace=False))
    return inputs.from_edges(n, np.concatenate([rng.choice(dst, n_active), np.roll(dst, 1)]),
                             np.concatenate([dst, dst]))


def _say(*a):
    print(*a, flush=True)


# start nodes around a run of 3,584; one source, a repeated one, all 32; one
# step, and walks of many steps that share sorts
@pytest.mark.parametrize("n_active", [1, 511, 3583, 3584, 3585])
@pytest.mark.parametrize("k, R, L, c", [(1, 3, 1, 0.6), (2, 40, 255, 0.95), (32, 25, 64, 0.6)])
def test_plain_runs(n_active, k, R, L, c):
    _say(f"tuple runs: {n_active} start nodes, k={k} R={R} L={L} c={c}")
    g = _graph(n_active)
    src = [int(v) for v in np.random.Generator(np.random.PCG64(k)).integers(0, g.n, k)]
    src[-1] = src[0]
    G = S.load_csr(g)
    sums, st = S.simrank_tuple_meets(G, [S.make_query(s, c=c, eps=0.5, seed=9, walk_cap=L, R=R) for s in src])
    steps = O.walk_table_plain(g, 9, c, L, np.repeat(np.flatnonzero(g.in_degree() > 0), R).astype(np.int32),
                               np.tile(np.arange(R, dtype=np.uint32), n_active))[1]
    assert st.moves == int(steps.sum())
    for q, s in enumerate(src):
        assert np.array_equal(sums[q], O.meet_counts_plain(g, s, 9, c, L, R).astype(np.uint64)), (q, s)
    G.free()


@pytest.mark.parametrize("n_active", [1, 3585])
def test_stratified_runs(n_active):
    _say(f"stratified tuple runs: {n_active} start nodes")
    g = _graph(n_active)
    G = S.load_csr(g)
    s = int(np.flatnonzero(g.in_degree() > 0)[0])
    qs = [S.make_stratified_query(v, c=0.6, eps=0.5, seed=9, z=30, phi=20) for v in (s, 0)]
    sums, _ = S.simrank_tuple_meets(G, qs)
    P = O.strat_params(g.n, 0.6, 0.5, z=30.0, phi=20)
    for q, v in enumerate((s, 0)):
        assert np.array_equal(sums[q], O.strat_sums(g, v, 9, P)), q
    G.free()
