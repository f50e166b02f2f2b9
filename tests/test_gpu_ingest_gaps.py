"""Loading graphs with many rows without edges between the edges of a tile: each
edge must come to its own row, and the load must not go through such rows one
block at a time.
"""
import time

import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu


FEW = 1 << 20     # edges up to which tiles are of 1,024, beyond it of 4,096


def _gap(rows, m, seed, where=1, front=0):
    """m edges in four rows, `rows` rows without any behind row number `where`;
    `front` edges more in a row in front."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = rows + 5
    at = [1 + (i if i <= where else i + rows) for i in range(4)]
    deg = np.zeros(n, np.int64)
    deg[0] = front
    deg[at] = m // 4
    deg[at[3]] += m - 4 * (m // 4)
    m += front
    off = np.concatenate([[0], np.cumsum(deg)])
    return inputs.CSR(n, off.astype(np.int32), rng.choice(at, m).astype(np.int32)), at


# rows per edge around the most that are gone through (16, edges counted as 256 at
# least); one tile of edges, and a second one that starts inside the last rows;
# both sizes of tiles
@pytest.mark.parametrize("front, tile", [(0, 1024), (FEW, 4096)])
@pytest.mark.parametrize("m", [4, 255, 257, 1024, 1030, 4096, 4100, 9000])
@pytest.mark.parametrize("around", [-8, 0, 1, 3000])
def test_rows_behind_a_gap_equal_oracle(m, around, front, tile):
    rows = 16 * min(max(m, 256), tile) + around
    print(f"gap: {rows} rows, {m} edges behind {front}", flush=True)
    g, at = _gap(rows, m, rows, front=front)
    G = S.load_csr(g)
    vs = np.array(at + [2, g.n - 2], np.int32)
    cnt = S.simrank_single_source_ex(G, S.make_query(at[1], seed=3, R=300, walk_cap=16))[1]
    assert np.array_equal(cnt[vs], O.meet_counts_plain(g, at[1], 3, 0.6, 16, 300, vs))
    vs = np.repeat(np.array(at, np.int32), 50)
    js = np.tile(np.arange(50, dtype=np.uint32), 4)
    paths, lens = S.simrank_walks(G, S.make_query(at[0], seed=5, R=50, walk_cap=8), vs, js)
    for i in range(0, 200, 7):
        for t in range(lens[i]):
            v, u = paths[i][t], paths[i][t + 1]
            assert u in g.in_src[g.in_off[v]:g.in_off[v + 1]]
    G.free()


# Rows around the edges of the large tiles (of the small ones where there are no
# more edges), as walks and pool sizes see them.
@pytest.mark.parametrize("front, tile", [(0, 1024), (FEW, 4096), (FEW - 4096, 1024)])
@pytest.mark.parametrize("behind", [(-1, 0), (0, 0), (1, 0), (7, 2), (0, 900)])
def test_rows_around_tiles_equal_oracle(front, tile, behind):
    more, empty = behind
    deg = [front] + [0] * empty + [tile + more, 3, 0] + [0] * empty + [1, 2 * tile - 4 + more, 0, 5]
    print(f"rows: {deg[0]} edges in front, tiles of {tile}, {behind}", flush=True)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    src = np.random.Generator(np.random.PCG64(3)).integers(0, len(deg), off[-1]).astype(np.int32)
    g = inputs.CSR(len(deg), off, src)
    G = S.load_csr(g)
    act = np.flatnonzero(g.in_degree() > 0)
    v, j = np.repeat(act, 400).astype(np.int32), np.tile(np.arange(400, dtype=np.uint32), act.size)
    paths, lens = S.simrank_walks(G, S.make_query(0, seed=3, walk_cap=8, R=400), v, j)
    opaths, olens = O.walk_table_plain(g, 3, 0.6, 8, v, j)
    assert np.array_equal(paths, opaths) and np.array_equal(lens, olens)
    assert S.simrank_build_index(G, seg_log2=1, kappa=0.5, c=0.6, seed=1)["segments"] == int(O.pool_sizes(g, 0.5).sum())
    G.free()


# The same rows and edges with the gap inside the tile and behind all edges; gone
# through by one block the first takes twice as long.
def test_a_gap_is_not_gone_through_by_one_block():
    def least(where):
        g, _ = _gap(1 << 23, 1000, 1, where)
        best = 1e9
        for _ in range(5):
            t = time.perf_counter()
            S.load_csr(g).free()
            best = min(best, time.perf_counter() - t)
        return best
    inside, behind = least(1), least(3)
    print(f"gap: {inside * 1e3:.2f} ms inside, {behind * 1e3:.2f} behind", flush=True)
    assert inside < 1.4 * behind
