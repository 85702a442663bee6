"""The column search where it is known to run: counts whose instrumented runs say
how many roots went whole, how many units there were, split by a second and a
third column, left to the row search, and searched by the deep run.  Exact counts
against closed forms, the global-set path, and the search from the other side."""
import ctypes
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu

WORK = ["whole", "units", "split2", "split3", "left", "children", "n_long"]


@pytest.fixture(scope="module")
def bc():
    from paper_2403_07858_amd import bc as m
    return m


def work(bc):
    a = (ctypes.c_uint64 * len(WORK))()
    bc._lib.bcint_last_columns(a)
    return dict(zip(WORK, a))


def complete(a, b):
    us, vs = np.divmod(np.arange(a * b), b)
    return gg.graph_from_pairs(a, b, us, vs)


# roots of more than 64 neighbours, whole (out of the slab) and by units; units
# split by one and two more columns; lists that fill up; units past 128 columns,
# which only the deep run takes
@pytest.mark.parametrize("a,b,p,q,reached", [
    (2300, 100, 3, 2, ["whole"]), (300, 64, 5, 3, ["whole"]), (300, 64, 5, 4, ["units"]),
    (300, 64, 6, 5, ["split2"]), (300, 64, 6, 7, ["split2", "split3"]), (400, 40, 5, 7, ["split3"]),
    (150, 200, 6, 3, ["split2"]), (150, 200, 6, 4, ["split3", "n_long"]), (500, 150, 5, 3, ["split2", "n_long"]),
    (500, 150, 5, 4, ["split3", "n_long"]), (500, 150, 6, 4, ["split3", "n_long"])])
def test_complete_graphs(bc, a, b, p, q, reached):
    G = bc.build_graph(complete(a, b))
    U = bc.BC_ANCHOR_U
    want = comb(a, p) * comb(b, q)
    assert bc.bc_count(G, p, q, anchor=U, instrument=True) == want
    w = work(bc)
    print(a, b, (p, q), w, flush=True)
    assert all(w[x] for x in reached), w
    assert bc.bc_count(G, p, q, anchor=U) == want
    assert bc.bc_count(G, p, q, anchor=U, timeout_ms=60_000) == want   # the kernels that watch the clock
    G.close()


# dense graphs whose units are long and many: by units left to the row search one
# by one these ran for many seconds
@pytest.mark.parametrize("a,b,p,q", [(200, 70, 6, 7), (200, 150, 6, 4), (200, 200, 6, 4), (1000, 150, 4, 4)])
def test_dense_graphs_end(bc, a, b, p, q):
    G = bc.build_graph(complete(a, b))
    assert bc.bc_count(G, p, q, anchor=bc.BC_ANCHOR_U, timeout_ms=3500) == comb(a, p) * comb(b, q)   # 0.1 to 0.7 s
    G.close()


RANDOM = {
    "er": (lambda: gg.er_bipartite(3000, 200, 120_000, seed=34), [(3, 3, "whole", "units"), (3, 4, "units", "left")]),
    "hubs": (lambda: gg.chung_lu_bipartite(1500, 1500, 100_000, 2.4, 2.4, 700, 700, seed=39),
             [(4, 4, "whole", "units", "left"), (4, 6, "units", "left"), (5, 5, "units"), (6, 6, "split2"),
              (5, 7, "split2", "left"), (6, 7, "split2", "split3", "left")]),
    "wide": (lambda: gg.chung_lu_bipartite(3000, 300, 60_000, 2.3, 2.3, 250, 2000, seed=31),
             [(4, 4, "whole", "left"), (5, 5, "whole", "units"), (4, 7, "split2", "left"), (6, 6, "split2")]),
}


@pytest.mark.parametrize("name", sorted(RANDOM))
def test_random_graphs(bc, name):
    make, queries = RANDOM[name]
    G = bc.build_graph(make())
    U, V = bc.BC_ANCHOR_U, bc.BC_ANCHOR_V
    for p, q, *reached in queries:
        want = bc.bc_count(G, p, q, anchor=U, instrument=True)
        w = work(bc)
        print(name, (p, q), want, w, flush=True)
        assert want > 0 and all(w[x] for x in reached), w
        assert bc.bc_count(G, p, q, anchor=V) == want
        assert bc.bc_count(G, p, q, anchor=U, roots_per_wave=1, waves_per_cu=2) == want
        assert bc.bc_count(G, p, q, anchor=U, timeout_ms=60_000) == want
        if p <= 4 and q <= 4:
            assert bc.bc_count(G, p, q, anchor=U, sets=bc.BC_SETS_SORTED) == want
        # shorter lists: what is split and left moves
        assert bc.bc_count(G, p, q, anchor=U, scratch_cap_bytes=192 << 20) == want
    G.close()
