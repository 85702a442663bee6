"""The candidate pass (k_root_build): roots counted in small blocks, those too
large for them in large ones, by id ranges, and in the dense array past that.
Exact counts against closed forms and the oracle at the sizes where one takes
over from the next and where the rows no longer fit what is built at once."""
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


# a around the small blocks' limits (1500, 1800, 2048), the rows of a large
# block (3072 words), its id ranges' candidates (4096) and its table (8192); b
# at one row word, two and three
@pytest.mark.parametrize("a,b", [(1502, 3), (1503, 64), (1800, 65), (1802, 4), (2050, 130), (3074, 64), (3074, 65),
                                 (4099, 5), (4099, 66), (8194, 4), (8330, 65)])
def test_complete_graphs(bc, a, b):
    G = bc.build_graph(complete(a, b))
    for p, q in [(2, 2), (2, 3), (3, 2), (3, 3)]:
        want = comb(a, p) * comb(b, q)
        print(f"K_{{{a},{b}}} ({p},{q})", flush=True)
        assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U) == want, (a, b, p, q)
        assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, waves_per_cu=1) == want, (a, b, p, q)
        # subsets whose first vertex is among the first half
        half = a // 2
        got = bc.bc_count_roots(G, p, q, bc.BC_ANCHOR_U, 0, half)
        assert got == want - comb(a - half, p) * comb(b, q), (a, b, p, q)
    G.close()


@pytest.mark.parametrize("n_u,n_v,m", [(20_000, 20, 90_000), (9_000, 24, 60_000), (6_000, 150, 60_000),
                                       (3_000, 200, 60_000)])
def test_random_graphs(bc, n_u, n_v, m):
    g = gg.chung_lu_bipartite(n_u, n_v, m, 2.5, 2.5, n_v * 0.9, n_u * 0.6, seed=5)
    G = bc.build_graph(g)
    for p, q in [(2, 3), (2, 4), (3, 3), (3, 4)]:
        want = oracle.count(g, p, q, anchor="V")
        print(n_u, n_v, (p, q), want, flush=True)
        assert want > 0
        assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U) == want
        assert bc.bc_count(G, p, q, scratch_cap_bytes=bc.bc_scratch_estimate(G, p, q)) == want
    G.close()
