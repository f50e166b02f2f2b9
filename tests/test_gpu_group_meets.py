"""Query groups whose walks meet often: most lanes of a wave meet members at one
step, several members at once.

Counts and weighted sums are integers and must equal the lone queries' and the CPU
oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu

ISEED = 9


def _star(n):      # every node's one in-neighbour is node 0
    return inputs.CSR(n, np.arange(n + 1, dtype=np.int32), np.zeros(n, np.int32))


def _cycle(n):     # walks from different nodes never meet; a source's own is met all along
    return inputs.CSR(n, np.arange(n + 1, dtype=np.int32), np.roll(np.arange(n), 1).astype(np.int32))


GRAPHS = {"star": _star(70), "dense": inputs.erdos_renyi_in(20, 6.0, seed=1),
          "small": inputs.erdos_renyi_in(150, 4.0, seed=2), "two": _cycle(2)}


# one member of an instance, its most and one more; all members of one source
# among the others
@pytest.mark.parametrize("members", [2, 8, 9, 32])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_frequent_meets_equal_lone_and_oracle(name, members):
    print(f"group meets: {name}, {members} members", flush=True)
    g, R, rng = GRAPHS[name], 400, np.random.default_rng(members)
    G = S.load_csr(g)
    S.simrank_build_index(G, seg_log2=1, kappa=1.0, c=0.6, seed=ISEED)
    src = [int(s) for s in rng.integers(0, g.n, members)]
    src[-1] = src[0]
    plan = S.BatchPlan([G], [S.make_query(s, seed=3, R=R) for s in src] +
                       [S.make_query(s, seed=3, R=R, mode=S.MODE_STITCHED) for s in src] +
                       [S.make_stratified_query(s, eps=0.2, seed=6, z=300, phi=9) for s in src])
    assert plan.n_groups == 3
    for _ in range(2):
        plan.run()
        plan.wait()
        for i in {0, members // 2, members - 1}:
            s = src[i]
            lone = [S.simrank_single_source_ex(G, S.make_query(s, seed=3, R=R, mode=m))[1]
                    for m in (S.MODE_PLAIN, S.MODE_STITCHED)]
            assert np.array_equal(plan.read(i)[1], lone[0])
            assert np.array_equal(plan.read(i)[1], O.meet_counts_plain(g, s, 3, 0.6, 64, R))
            assert np.array_equal(plan.read(members + i)[1], lone[1])
            strat = S.simrank_single_source_stratified(G, S.make_stratified_query(s, eps=0.2, seed=6, z=300, phi=9))
            assert np.array_equal(plan.read_stratified(2 * members + i)[2], strat[2])
    plan.free()
    G.free()


# A group walks once for all its members, so it takes a fraction of what they take
# without it, also where meets are frequent: of 32 members 0.38 of their time, and
# 1.03 with the meets of a step taken one lane after another.
def test_frequent_meets_leave_the_group_faster():
    G = S.load_csr(inputs.erdos_renyi_in(1000, 5.0, seed=1))

    def least(groups):
        plan = S.BatchPlan([G], [S.make_query(i, seed=3, R=9502) for i in range(32)], groups=groups)
        best = 1e9
        for _ in range(9):
            plan.run()
            best = min(best, plan.wait().ms)
        plan.free()
        return best
    group, lone = least(True), least(False)
    print(f"group meets: {group:.3f} ms, ungrouped {lone:.3f}", flush=True)
    assert group < 0.63 * lone
    G.free()
