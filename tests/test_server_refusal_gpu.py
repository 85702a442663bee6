"""The service's refusals price a count by the searches that it takes: one that
ends in milliseconds by columns is not refused by what its rows would take."""
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def test_counts_by_columns_are_not_refused():
    from paper_2403_07858_amd import bc

    small = bc.build_graph(gg.chung_lu_bipartite(2000, 1000, 16000, 2.2, 2.2, 150, 150, seed=40))
    srv = bc.Server(max_inflight=1, max_batch=1)
    sid = srv.add_graph(small)
    for m, p, q in [(120_000, 6, 6), (300_000, 6, 6), (300_000, 4, 4), (300_000, 5, 5)]:
        G = bc.build_graph(gg.chung_lu_bipartite(m // 20, m // 40, m, 2.1, 2.1, m // 187, m // 187, seed=3))
        gid = srv.add_graph(G)
        # a served count of that depth, by rows: the rate that rows are priced at
        st, _, _ = srv.poll(srv.submit(sid, p, q))
        assert st == bc.BC_OK
        want = bc.bc_count(G, p, q)   # 3 to 24 ms
        st, val, info = srv.poll(srv.submit(gid, p, q, deadline_ns=srv.now_ns() + 2_000_000_000))
        print(m, (p, q), bc.bc_status_string(st), info, flush=True)
        assert st == bc.BC_OK and val == want
    srv.close()
