"""Device memory of a loaded graph: rows packed in 4 bytes are kept only where
queries can read them.
"""
import numpy as np
import pytest

from paper_2304_04015_amd import simrank as S
from test_gpu_packed import _graph

pytestmark = pytest.mark.gpu


# no hubs; as many hubs as a kernel has rows for, and one more
@pytest.mark.parametrize("slots, hubs, hub_deg, packed", [
    (4000, 0, 0, True), (4194305, 6848, 512, True), (4194305, 6849, 512, False)])
def test_packed_rows_take_memory_only_where_read(slots, hubs, hub_deg, packed):
    print(f"memory: {slots} slots, {hubs} nodes of in-degree {hub_deg}", flush=True)
    g = _graph(slots, hubs, hub_deg, slots + hubs)
    G = S.load_csr(g)
    info = G.info()
    # rows (8 bytes a slot) and nodes (4), per node its row, its place among the
    # nodes with in-edges and its out-degree
    base = 12 * slots + 12 * g.n + 4 * info["n_active"]
    extra = 4 * slots + 8 * hubs if packed else 0
    assert base + extra <= info["device_bytes"] <= base + extra + 4 * 256
    G.free()


def test_falling_offsets_are_refused_at_the_first_such_row():
    off = np.array([0, 3, 2, 1, 4], np.int32)
    with pytest.raises(S.SimRankError, match="decreases at row 1"):
        S.simrank_load_graph(4, off, np.zeros(4, np.int32))
