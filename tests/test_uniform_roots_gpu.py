"""Dense and random graphs, whose roots' rows are all about the same length: the
plan weighs the subsets of their columns against those of their rows.  Exact
counts from both sides, and time limits that the dearer search would pass."""
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,b,p,q,ms", [(1000, 64, 4, 6, 150), (400, 64, 5, 7, 250), (1000, 100, 4, 4, 150), (400, 100, 5, 5, 250)])
def test_complete_graphs(a, b, p, q, ms):
    from paper_2403_07858_amd import bc

    us, vs = np.divmod(np.arange(a * b), b)
    G = bc.build_graph(gg.graph_from_pairs(a, b, us, vs))
    want = comb(a, p) * comb(b, q)
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U) == want
    # by rows 5, 44, 10 and 35 ms; by columns 300, 550, 18 and 50
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, timeout_ms=ms) == want
    G.close()


@pytest.mark.parametrize("n_u,n_v,fill,p,q", [(1500, 500, 0.2, 5, 7), (2500, 200, 0.3, 4, 6), (400, 100, 0.5, 5, 7)])
def test_random_graphs(n_u, n_v, fill, p, q):
    from paper_2403_07858_amd import bc

    G = bc.build_graph(gg.er_bipartite(n_u, n_v, int(n_u * n_v * fill), seed=5))
    want = bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U)
    assert want > 0
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, root_build=bc.BC_ROOT_BUILD_TWO_PASS) == want
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, scratch_cap_bytes=160 << 20) == want
    G.close()
