"""Units of served requests claimed by subtraction: requests of fewer units than
the grid has blocks (most blocks come too late), of one and of several units per
claim, entries used again by requests of every kind while kernels run.

Counts and weighted sums are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

ISEED = 9


@pytest.mark.parametrize("n, slots", [(2, 1), (60, 2), (700, 3), (3000, 16)])
def test_every_unit_is_taken_once(n, slots):
    print(f"ring: n={n}, {slots} in flight", flush=True)
    g = inputs.erdos_renyi_in(n, 3.0, seed=n)
    G = S.load_csr(g)
    S.simrank_build_index(G, seg_log2=1, kappa=1.0, c=0.6, seed=ISEED)
    Q, P = O.pool_sizes(g, 1.0), O.strat_params(n, 0.6, 0.1, 200, 12)
    rng = np.random.Generator(np.random.PCG64(n))
    srv = S.Server(G, max_slots=slots, max_R=2000, max_L=64)
    sent = []
    for i in range(36):
        s, R, kind = int(rng.integers(0, n)), int(rng.choice([1, 40, 2000])), i % 3
        q = (S.make_stratified_query(s, eps=0.1, seed=i, z=200, phi=12) if kind == 2 else
             S.make_query(s, seed=i, R=R, mode=S.MODE_STITCHED if kind else S.MODE_PLAIN))
        sent.append((srv.submit(q), s, R, kind, i))
    vs = np.unique(np.r_[0:min(n, 40), n - 1]).astype(np.int32)
    for t, s, R, kind, i in sent:
        if kind == 2:
            got, want = srv.wait_stratified(t)[2], O.strat_sums(g, s, i, P, vs)
        elif kind == 1:
            got, want = srv.wait(t)[1], O.meet_counts_stitched(g, s, i, ISEED, 0.6, 64, 2, Q, R, vs)
        else:
            got, want = srv.wait(t)[1], O.meet_counts_plain(g, s, i, 0.6, 64, R, vs)
        assert np.array_equal(got[vs], want), (i, s, R, kind)
    srv.destroy()
    G.free()
