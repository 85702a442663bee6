"""The column search when memory is short: its buffers come on top of the row
search's, so a count that fits without them has to finish by rows."""
import pytest

from paper_2403_07858_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bc():
    from paper_2403_07858_amd import bc as m
    return m


@pytest.fixture(scope="module")
def graph(bc):
    from test_column_limits_gpu import hub_and_sparse_rows

    G = bc.build_graph(hub_and_sparse_rows(1000, 800, 100, seed=4))
    yield G
    G.close()


class Limited:
    """Allocator hook that refuses its call number `fail_at`, and what would take
    it past `limit` live bytes."""

    def __init__(self, bc, limit=None, fail_at=None):
        import torch

        self.torch, self.limit, self.live, self.now, self.peak = torch, limit, {}, 0, 0
        self.fail_at, self.calls = fail_at, 0
        self.hook = bc.Allocator(self.alloc, self.free)

    def alloc(self, n, stream):
        self.calls += 1
        if self.calls - 1 == self.fail_at or (self.limit is not None and self.now + n > self.limit):
            return 0
        t = self.torch.empty(n, dtype=self.torch.uint8, device="cuda")
        self.live[t.data_ptr()] = t
        self.now += n
        self.peak = max(self.peak, self.now)
        return t.data_ptr()

    def free(self, p, stream):
        self.torch.cuda.synchronize()
        self.now -= self.live.pop(p).numel()


def test_hook_short_of_the_columns(bc, graph):
    U = bc.BC_ANCHOR_U
    want = bc.bc_count(graph, 5, 4, anchor=U, sets=bc.BC_SETS_SORTED)
    free = Limited(bc)
    assert bc.bc_count(graph, 5, 4, anchor=U, allocator=free.hook) == want
    print("peak", free.peak, flush=True)
    short = Limited(bc, free.peak - 1)
    assert bc.bc_count(graph, 5, 4, anchor=U, allocator=short.hook) == want
    assert short.peak < free.peak and not short.live
    # one refusal at a time: the search's own blocks (the columns, the slabs
    # beside them) have a second try without columns, the rest end the call
    done = []
    for k in range(free.calls):
        al = Limited(bc, fail_at=k)
        try:
            assert bc.bc_count(graph, 5, 4, anchor=U, allocator=al.hook) == want
            done.append(k)
        except bc.BCError as e:
            assert e.status == bc.BC_E_OOM
        assert not al.live, k
    print("allocations", free.calls, "done without", done, flush=True)
    assert len(done) >= 6 and done == list(range(done[0], free.calls))


@pytest.mark.parametrize("opts", [{}, {"split_rows": 64}, {"split_rows": 64, "root_build": 1}])
def test_caps(bc, graph, opts):
    # a larger cap never refuses what a smaller one took
    U = bc.BC_ANCHOR_U
    want = bc.bc_count(graph, 5, 4, anchor=U)
    fits, caps = False, []
    cap = 24 << 20
    while cap < 400 << 20:
        try:
            got, st = bc.bc_count(graph, 5, 4, anchor=U, scratch_cap_bytes=cap, with_stats=True, **opts)
            assert got == want and st["scratch_bytes"] <= cap
            fits = True
        except bc.BCError as e:
            assert e.status == bc.BC_E_OOM
            assert not fits, (cap, caps)
        caps.append((cap, fits))
        print(opts, cap >> 10, fits, flush=True)
        cap = int(cap * 1.07)
    assert fits
