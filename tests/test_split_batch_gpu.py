"""Batches with the runtime split on: a wavefront goes from the tasks of one job
to the queued subtasks of any other, whose leaf values are not the same."""
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


# jobs of one depth and twelve different q, so that every pair of job numbers
# meets on some wavefront; few wavefronts, so that each runs many jobs
@pytest.mark.parametrize("waves", [1, 12])
@pytest.mark.parametrize("order", ["up", "down"])
def test_counts_equal_closed_forms(waves, order):
    from paper_2403_07858_amd import bc

    a, b, p = 44, 24, 5
    us, vs = np.divmod(np.arange(a * b), b)
    G = bc.build_graph(gg.graph_from_pairs(a, b, us, vs))
    qs = [2, 3, 4, 5, 6, 8, 9, 10, 7, 11, 12, 13]
    if order == "down":
        qs.reverse()
    U = bc.BC_ANCHOR_U
    vals, sts = bc.bc_count_batch([G] * len(qs), [p] * len(qs), qs, anchor=U, split_rows=4, switch_depth=2,
                                  waves_per_cu=waves)
    assert sts == [0] * len(qs)
    want = [comb(a, p) * comb(b, q) for q in qs]
    assert vals == want, [q for q, v, w in zip(qs, vals, want) if v != w]
    G.close()
