"""Row searches whose first candidates are shared out by their child rows: few
roots with wide rows that keep each other.  Exact counts against closed forms,
whole, by ranges of roots, on fewer wavefronts, under a cap and in a batch."""
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b,p,q", [(45, 300, 6, 6), (60, 300, 6, 5), (90, 300, 5, 5), (30, 300, 6, 6), (40, 70, 6, 8),
                                     (36, 130, 8, 7)])
def test_complete_graphs(a, b, p, q):
    from paper_2403_07858_amd import bc

    us, vs = np.divmod(np.arange(a * b), b)
    G = bc.build_graph(gg.graph_from_pairs(a, b, us, vs))
    want = comb(a, p) * comb(b, q)
    print(f"K_{{{a},{b}}} ({p},{q})", flush=True)
    U = bc.BC_ANCHOR_U
    assert bc.bc_count(G, p, q, anchor=U) == want
    assert bc.bc_count(G, p, q, anchor=U, waves_per_cu=4, roots_per_wave=3) == want
    assert bc.bc_count(G, p, q, anchor=U, split_rows=64) == want
    assert bc.bc_count(G, p, q, anchor=U, root_build=bc.BC_ROOT_BUILD_TWO_PASS) == want
    parts = [bc.bc_count_roots(G, p, q, U, lo, hi) for lo, hi in ((0, 3), (3, a // 2), (a // 2, a))]
    assert sum(parts) == want
    assert bc.bc_count(G, p, q, scratch_cap_bytes=bc.bc_scratch_estimate(G, p, q)) == want
    G2 = bc.build_graph(gg.graph_from_pairs(a, b, us, vs))
    vals, sts = bc.bc_count_batch([G, G2], [p, p], [q, q])
    assert sts == [0, 0] and vals == [want, want]
    G.close()
    G2.close()
