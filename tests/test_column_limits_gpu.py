"""Roots at the widest the column search takes neighbour by neighbour: sparse
rows over 1023, 1024 and 1025 neighbours, whose last column is that of the
lowest-ranked neighbour.  Exact counts against the global-set path."""
import ctypes

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def hub_and_sparse_rows(n, rows, shared, seed):
    """Vertex 0 of U has n neighbours; `rows` others share a fifth to nine fifths
    of `shared` of them each and have as many neighbours in all (the rest their
    own), so that they rank behind vertex 0 and are its candidates."""
    us, vs = [np.zeros(n, dtype=np.int64)], [np.arange(n, dtype=np.int64)]
    for r in range(rows):
        common = shared * (1 + 2 * (r % 5)) // 5
        pick = np.argsort(gg.draws_u64(seed, r, 0, n), kind="stable")[:common]
        us.append(np.full(n, r + 1, dtype=np.int64))
        vs.append(np.concatenate([pick, n + r * n + np.arange(n - common)]))
    return gg.graph_from_pairs(rows + 1, n + rows * n, np.concatenate(us), np.concatenate(vs))


@pytest.mark.parametrize("n", [1022, 1023, 1024, 1025])
def test_widest_unit_roots(n):
    from paper_2403_07858_amd import bc

    g = hub_and_sparse_rows(n, 800, 100, seed=3)
    G = bc.build_graph(g)
    p, q = 5, 4
    # the global-set path shares neither search with the counts checked
    want = bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, sets=bc.BC_SETS_SORTED)
    print(n, (p, q), want, flush=True)
    assert want > 0
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U) == want
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_V) == want
    # the roots' first units are those of their lowest-ranked neighbour
    work = (ctypes.c_uint64 * 7)()
    assert bc.bc_count_roots(G, p, q, bc.BC_ANCHOR_U, 0, 400, instrument=True) <= want
    bc._lib.bcint_last_columns(work)
    print("units", work[1], flush=True)
    assert (work[1] > 0) == (n <= 1023)
    G.close()
