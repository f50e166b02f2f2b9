"""Packing of a query group's source walks (blocks of member positions per step,
padded to 16 bytes) and the group compare that reads them: every member's counts
must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu


# members around the half wave, the four-word pieces and the two tile shapes;
# walk counts around a packing block of 32 (ragged between members: shorter
# members have no walk j), a walk cap of one step and the longest one
@pytest.mark.parametrize("members", [2, 3, 4, 5, 8, 9, 31, 32])
@pytest.mark.parametrize("R, L, c", [(1, 1, 0.6), (33, 255, 0.96), (700, 20, 0.6)])
def test_group_counts_equal_oracle(members, R, L, c):
    print(f"group of {members}: R={R} L={L} c={c}", flush=True)
    g = inputs.erdos_renyi_in(90, 3.0, seed=members)
    G = S.load_csr(g)
    # sources with and without in-edges; a repeated one; ragged walk counts
    src = [int(v) for v in np.random.Generator(np.random.PCG64(R)).integers(0, g.n, members)]
    src[-1] = src[0]
    Rs = [max(1, R - 5 * (i % 7)) for i in range(members)]
    qs = [S.make_query(s, c=c, eps=0.5, seed=5, walk_cap=L, R=r) for s, r in zip(src, Rs)]
    plan = S.BatchPlan([G], qs)
    assert plan.n_groups == 1
    plan.run()
    plan.wait()
    for i, (s, r) in enumerate(zip(src, Rs)):
        _, cnt = plan.read(i)
        assert np.array_equal(cnt, O.meet_counts_plain(g, s, 5, c, L, r)), (i, s, r)
    plan.free()
    G.free()
