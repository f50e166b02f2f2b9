"""Units of served requests claimed several at once: requests of many more units than
the grid has blocks (units of one node), so that claims take runs of two to four,
shorten towards a request's end and reach past it, while entries are used again by
requests of every kind.

Counts and weighted sums are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

ISEED = 9


# a claim takes min(4, units left / 512) units: around the least that take two and
# four, several tiles, and many
@pytest.mark.parametrize("n, R, slots", [(1023, 300, 2), (1026, 300, 3), (2100, 300, 2), (1300, 9000, 3), (6000, 40, 16)])
def test_runs_of_units_are_taken_once(n, R, slots):
    print(f"ring runs: n={n} R={R}, {slots} in flight", flush=True)
    rng = np.random.Generator(np.random.PCG64(n))
    dst = np.arange(n)                                    # every node has in-edges: n units a tile
    g = inputs.from_edges(n, np.concatenate([rng.integers(0, n, n), np.roll(dst, 1)]), np.concatenate([dst, dst]))
    G = S.load_csr(g)
    S.simrank_set_tuning(G, 1, 0)
    S.simrank_build_index(G, seg_log2=1, kappa=1.0, c=0.6, seed=ISEED)
    Q, P = O.pool_sizes(g, 1.0), O.strat_params(n, 0.6, 0.1, 200, 12)
    srv = S.Server(G, max_slots=slots, max_R=max(R, 2000), max_L=64)
    sent = []
    for i in range(24):
        s, r, kind = int(rng.integers(0, n)), int(rng.choice([1, R])), i % 3
        q = (S.make_stratified_query(s, eps=0.1, seed=i, z=200, phi=12) if kind == 2 else
             S.make_query(s, seed=i, R=r, mode=S.MODE_STITCHED if kind else S.MODE_PLAIN))
        sent.append((srv.submit(q), s, r, kind, i))
    vs = np.unique(np.linspace(0, n - 1, 60).astype(np.int32))
    for t, s, r, kind, i in sent:
        if kind == 2:
            got, want = srv.wait_stratified(t)[2], O.strat_sums(g, s, i, P, vs)
        elif kind == 1:
            got, want = srv.wait(t)[1], O.meet_counts_stitched(g, s, i, ISEED, 0.6, 64, 2, Q, r, vs)
        else:
            got, want = srv.wait(t)[1], O.meet_counts_plain(g, s, i, 0.6, 64, r, vs)
        assert np.array_equal(got[vs], want), (i, s, r, kind)
    srv.destroy()
    G.free()
