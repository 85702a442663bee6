"""The column search (k_columns): roots counted by the other side's subsets,
whole, neighbour by neighbour, or split by a second neighbour, with the row
search over what it leaves.  Every count against a closed form or the oracle,
exactly, at the sizes where its tiles, tuple tables and word counts end."""
from math import comb

import numpy as np
import pytest

import oracle
from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bc():
    from paper_2403_07858_amd import bc as m
    return m


def complete(a, b):
    us, vs = np.divmod(np.arange(a * b), b)
    return gg.graph_from_pairs(a, b, us, vs)


# candidates around the words a column is searched in (2, 8, 16, 24, 40 and past
# them), neighbours around the column counts (a tuple more or less than a
# round, and the ends of the tables of five, four, three and two)
@pytest.mark.parametrize("a,b", [(65, 7), (66, 27), (120, 28), (129, 29), (130, 41), (260, 12), (513, 10), (514, 13),
                                 (770, 9), (1030, 11), (1540, 8), (1600, 6), (2570, 7), (140, 64), (100, 65),
                                 (90, 127), (80, 129), (70, 200)])
def test_complete_graphs(bc, a, b):
    G = bc.build_graph(complete(a, b))
    for p, q in [(3, 2), (3, 3), (3, 6), (4, 3), (4, 4), (4, 5), (5, 5), (5, 6), (6, 4), (6, 6), (4, 7), (6, 7)]:
        want = comb(a, p) * comb(b, q)
        if want >> 128 or (a > 2000 and p > 4):   # (past the search's words, minutes by rows)
            continue
        print(f"K_{{{a},{b}}} ({p},{q})", flush=True)
        got = bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U)
        assert got == want, (a, b, p, q, got, want)
    G.close()


SHAPES = {
    # name: (n_u, n_v, edges, queries counted by the oracle from the V side)
    "wide": (1500, 22, 14000, [(3, 3), (4, 4), (5, 4), (6, 5), (4, 6)]),
    "mid": (420, 60, 6000, [(3, 3), (3, 5), (4, 4), (5, 5), (4, 6)]),
    "square": (150, 150, 3400, [(3, 3), (4, 4), (5, 5), (6, 6), (6, 4), (4, 7)]),
}


@pytest.fixture(scope="module", params=sorted(SHAPES))
def shape(request, bc):
    n_u, n_v, m, queries = SHAPES[request.param]
    g = gg.chung_lu_bipartite(n_u, n_v, m, 2.6, 2.6, n_v * 0.9, n_u * 0.7, seed=31)
    return g, bc.build_graph(g), queries


def test_against_oracle(bc, shape):
    g, G, queries = shape
    for p, q in queries:
        want = oracle.count(g, p, q, anchor="U" if p <= q and g.n_u < 1000 else "V")
        print(g.n_u, g.n_v, (p, q), want, flush=True)
        assert want > 0
        for anchor in (bc.BC_ANCHOR_U, bc.BC_ANCHOR_V):
            assert bc.bc_count(G, p, q, anchor=anchor) == want, (p, q, anchor)
        # the routes that choose between the searches differently
        assert bc.bc_count(G, p, q, root_build=bc.BC_ROOT_BUILD_TWO_PASS) == want
        assert bc.bc_count(G, p, q, roots_per_wave=1, waves_per_cu=1) == want
        assert bc.bc_count_noalloc(G, p, q) == want
        est = bc.bc_scratch_estimate(G, p, q)
        got, st = bc.bc_count(G, p, q, with_stats=True, scratch_cap_bytes=est, instrument=True)
        assert got == want and st["scratch_bytes"] <= est
        half = g.n_u // 2
        parts = [bc.bc_count_roots(G, p, q, bc.BC_ANCHOR_U, lo, hi) for lo, hi in ((0, half), (half, g.n_u))]
        assert sum(parts) == want
    vals, sts = bc.bc_count_batch([G] * len(queries), [p for p, _ in queries], [q for _, q in queries])
    assert sts == [0] * len(queries)
    assert vals == [bc.bc_count(G, p, q) for p, q in queries]
