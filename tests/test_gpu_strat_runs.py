"""Preparation of the stratified kernel's pairs: 64 walks of a node at once, and
a slot's class from the run of slots it lies in.

Weighted sums are integers and must equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest

import oracle as O
from paper_2304_04015_amd import inputs
from paper_2304_04015_amd import simrank as S

pytestmark = pytest.mark.gpu


def _z_for(walks, phi):
    """The least integer z with `walks` walks per node or more (N grows with z)."""
    lo, hi = 1, 1 << 20
    while lo < hi:
        mid = (lo + hi) // 2
        if O.strat_params(100, 0.6, 0.1, mid, phi).N >= walks:
            hi = mid
        else:
            lo = mid + 1
    return lo


# around 64 walks; runs of 1, 2 and 4 slots (up to 4096 slots, 8192 and beyond);
# one class, two, and more classes of one slot than a run has slots
@pytest.mark.parametrize("walks", [1, 63, 64, 65, 129, 4096, 4097, 8192, 8193, 20001])
@pytest.mark.parametrize("phi", [1, 2, 48, 255])
def test_stratified_sums_equal_oracle(walks, phi):
    top = _z_for(walks, phi)
    for n, seed, z in ((100, 3, max(1, top - 1)), (331, 4, top)):
        P = O.strat_params(n, 0.6, 0.1, z, phi)
        print(f"stratified: N={P.N} phi={phi}", flush=True)
        g = inputs.erdos_renyi_in(n, 3.0, seed=seed)
        G = S.load_csr(g)
        s = int(np.flatnonzero(g.in_degree() > 0)[1])
        q = S.make_stratified_query(s, eps=0.1, seed=7, phi=phi, z=z)
        sums = S.simrank_single_source_stratified(G, q)[2]
        assert np.array_equal(sums, O.strat_sums(g, s, 7, P))
        G.free()
