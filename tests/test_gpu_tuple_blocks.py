"""Algorithm 2's tuple form with few start nodes, which take blocks of one wave.
Counts and weighted sums must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S
from test_gpu_tuple_runs import _graph

pytestmark = pytest.mark.gpu


# start nodes around a wave, the most of a small block (256) and half of it; walks
# per node around the large blocks that are resident (512); one source, a repeated
# one, all 32; one step, and walks of many steps that share sorts
@pytest.mark.parametrize("n_active", [1, 64, 65, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("k, R, L, c", [(1, 3, 1, 0.6), (2, 40, 255, 0.95), (32, 512, 16, 0.6), (3, 513, 32, 0.6)])
def test_few_start_nodes(n_active, k, R, L, c):
    print(f"tuple blocks: {n_active} start nodes, k={k} R={R} L={L} c={c}", flush=True)
    g = _graph(n_active)
    src = [int(v) for v in np.random.Generator(np.random.PCG64(k)).integers(0, g.n, k)]
    src[-1] = src[0]
    G = S.load_csr(g)
    sums, st = S.simrank_tuple_meets(G, [S.make_query(s, c=c, eps=0.5, seed=9, walk_cap=L, R=R) for s in src])
    steps = O.walk_table_plain(g, 9, c, L, np.repeat(np.flatnonzero(g.in_degree() > 0), R).astype(np.int32),
                               np.tile(np.arange(R, dtype=np.uint32), n_active))[1]
    assert st.moves == int(steps.sum())
    for q in range(min(k, 4)):
        assert np.array_equal(sums[q], O.meet_counts_plain(g, src[q], 9, c, L, R).astype(np.uint64)), (q, src[q])
    if k == 32:
        assert np.array_equal(sums[-1], sums[0])
    G.free()


@pytest.mark.parametrize("n_active", [1, 128, 256])
@pytest.mark.parametrize("z", [30, 900])
def test_few_start_nodes_stratified(n_active, z):
    print(f"tuple blocks, stratified: {n_active} start nodes, z={z}", flush=True)
    g = _graph(n_active)
    G = S.load_csr(g)
    s = int(np.flatnonzero(g.in_degree() > 0)[0])
    sums, _ = S.simrank_tuple_meets(G, [S.make_stratified_query(v, c=0.6, eps=0.5, seed=9, z=z, phi=20) for v in (s, 0)])
    P = O.strat_params(g.n, 0.6, 0.5, z=float(z), phi=20)
    for q, v in enumerate((s, 0)):
        assert np.array_equal(sums[q], O.strat_sums(g, v, 9, P)), q
    G.free()


# Long walks of 10 nodes against those of 300, which take a large block: 0.21 of
# their time, and 1.01 in large blocks too.
def test_few_start_nodes_take_less_time():
    def least(n):
        G = S.load_csr(inputs.erdos_renyi_in(n, 5.0, seed=1))
        q = S.make_query(0, c=0.95, eps=0.5, seed=3, walk_cap=255, R=2000)
        best = min(S.simrank_tuple_meets(G, [q])[1].ms for _ in range(7))
        G.free()
        return best
    few, many = least(10), least(300)
    print(f"tuple blocks: {few:.3f} ms, 300 start nodes {many:.3f}", flush=True)
    assert few < 0.6 * many
