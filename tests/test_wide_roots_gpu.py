"""The candidate pass's wide blocks: few roots of many wedges, and roots of tens
of thousands of neighbours.  Closed forms at the sizes where they take over from
the small and the large blocks, and where their table, id ranges and dense array do."""
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bc():
    from paper_2403_07858_amd import bc as m
    return m


def complete(a, b, hub=0):
    """K_{a,b}, and one more U vertex with `hub` neighbours of its own (in no
    biclique with the others, but the widest root)."""
    us, vs = np.divmod(np.arange(a * b), b)
    us = np.concatenate([us, np.full(hub, a)])
    vs = np.concatenate([vs, b + np.arange(hub)])
    return gg.graph_from_pairs(a + 1, b + hub, us, vs)


# few roots: past 4096 neighbours, 2^15 and 2^16 of them; more than 2^15 wedges a
# root on average; a hub of 2^15 neighbours (and one less, and past 2^16) beside
# roots at the small blocks' limits, the ranges' candidates and the table's size
@pytest.mark.parametrize("a,b,hub", [(7, 4095, 0), (7, 4097, 0), (30, 32767, 0), (30, 32768, 0), (12, 65537, 0),
                                     (300, 400, 0), (1100, 130, 0), (1802, 4, 32767), (1802, 4, 32768), (2050, 70, 40000),
                                     (4099, 66, 40000), (8330, 65, 70000)])
def test_closed_forms(bc, a, b, hub):
    G = bc.build_graph(complete(a, b, hub))
    U = bc.BC_ANCHOR_U
    for p, q in [(2, 2), (2, 3), (3, 2)]:
        want = comb(a, p) * comb(b, q)
        print(a, b, hub, (p, q), flush=True)
        assert bc.bc_count(G, p, q, anchor=U) == want
        assert bc.bc_count(G, p, q, anchor=U, waves_per_cu=1) == want
        assert bc.bc_count(G, p, q, anchor=U, scratch_cap_bytes=bc.bc_scratch_estimate(G, p, q)) == want
    # per vertex, attributed by this pass
    got = bc.bc_count_per_vertex(G, 2, 2, U)
    assert got == [(a - 1) * comb(b, 2)] * a + [0]
    G.close()
