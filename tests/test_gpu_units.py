"""Work units of the meet kernels (runs of nodes under tiles of source walks):
every (node, walk) pair must be counted exactly once, whatever the split.

Counts are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu


def _graph(n_active):
    """n_active nodes with one or two in-edges each, the nodes without any among them."""
    n = n_active + n_active // 3 + 2
    rng = np.random.Generator(np.random.PCG64(n_active))
    dst = np.sort(rng.choice(n, size=n_active, replace=False))
    return inputs.from_edges(n, np.concatenate([rng.integers(0, n, n_active), dst]),
                             np.concatenate([dst, np.roll(dst, 1)]))


# one node; around a unit of 256 nodes, a grid of 256 blocks, and two rounds of
# it; one tile of source walks, several with a small last one, and a tuned split
@pytest.mark.parametrize("n_active", [1, 2, 255, 256, 257, 513, 1500])
@pytest.mark.parametrize("R, L, vb", [(1, 8, 0), (700, 32, 0), (9000, 64, 0), (9000, 64, 100)])
def test_units_cover_every_pair_once(n_active, R, L, vb):
    g = _graph(n_active)
    print(f"units: {n_active} nodes with in-edges, R={R} L={L} nodes per unit {vb or 'auto'}", flush=True)
    s = int(np.flatnonzero(g.in_degree() > 0)[n_active // 2])
    G = S.load_csr(g)
    S.simrank_set_tuning(G, vb, 0)
    out, cnt, st = S.simrank_single_source_ex(G, S.make_query(s, seed=17, walk_cap=L, R=R))
    want, work = O.meet_counts_plain(g, s, 17, 0.6, L, R, with_work=True)
    assert np.array_equal(cnt, want)
    assert st.moves == int(work.sum())
    # the same query beside others in one launch: their units share the rounds
    qs = [S.make_query(s, seed=17 + i, walk_cap=L, R=max(1, R // (i + 1))) for i in range(3)]
    _, cnts, _ = S.simrank_batch([G], qs)
    assert np.array_equal(cnts[0], want)
    assert np.array_equal(cnts[2], O.meet_counts_plain(g, s, 19, 0.6, L, max(1, R // 3)))
    G.free()
