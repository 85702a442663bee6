"""Time limits inside the column search: a unit may run for a tenth of a second on
one wavefront, and stops at the limit all the same."""
import time
from math import comb

import numpy as np
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [0, 64 << 20])   # units split up, and with little room for that
def test_long_units_stop(cap):
    from paper_2403_07858_amd import bc

    a, b, p, q = 300, 64, 6, 7
    us, vs = np.divmod(np.arange(a * b), b)
    G = bc.build_graph(gg.graph_from_pairs(a, b, us, vs))
    opts = dict(anchor=bc.BC_ANCHOR_U, **({"scratch_cap_bytes": cap} if cap else {}))
    t = time.perf_counter()
    assert bc.bc_count(G, p, q, **opts) == comb(a, p) * comb(b, q)
    whole = time.perf_counter() - t   # some 0.4 s
    late = []
    for limit in (10, 20, 30):
        t = time.perf_counter()
        with pytest.raises(bc.BCError) as e:
            bc.bc_count(G, p, q, timeout_ms=limit, **opts)
        late.append((time.perf_counter() - t) * 1e3 - limit)
        assert e.value.status == bc.BC_E_TIMEOUT
    print("whole %.0f ms, late by" % (whole * 1e3), late, flush=True)
    # units of up to 150 ms were running; the clock is read every millisecond or so
    assert sorted(late)[1] < 40
    # a limit that is not reached changes nothing
    assert bc.bc_count(G, p, q, timeout_ms=60_000, **opts) == comb(a, p) * comb(b, q)
    G.close()
