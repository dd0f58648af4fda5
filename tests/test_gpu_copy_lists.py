"""Copy lists and page-table writes at the sizes where their way changes (GPU):
in the kernel arguments up to 128 copies and 512 row entries, by upload above
that and up to the 65,536 entries of a staging slot, rows cleared 128 at a time."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda", 0)


def _pool(pages, sessions, stride, cold="device"):
    from paper_2609_25782_amd.pool import HotColdPool
    return HotColdPool(1, 1, 64, "bf16", pages, pages, sessions, stride, cold_location=cold)


@pytest.mark.parametrize("cold", ["device", "host"])
@pytest.mark.parametrize("pages", [1, 127, 128, 129, 511, 512, 513, 2000])
def test_one_session_of_so_many_pages(dev, pages, cold):
    """Create (row write), evict dirty (copies), resume onto other pages (copies
    and row), extend by one page, destroy (row cleared)."""
    pool = _pool(2 * pages + 2, 2, 2 * pages + 2, cold)
    pool.set_host_copy(True)    # the copy kernel, also for the pinned-host tier
    words = pool.hot.view(torch.int32)
    words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
    ids = np.random.default_rng(pages).permutation(2 * pages + 2)[:pages]
    sid = pool.create_session(16 * pages - 3, [int(x) for x in ids])
    assert pool.page_table[sid, :pages].cpu().numpy().tolist() == ids.tolist()
    before = pool.hot_page_bytes(ids).cpu()
    pool.evict(sid)
    assert (pool.page_table[sid].cpu() == -1).all()
    pool.hot.zero_()
    pool.resume(sid)
    hot = pool.info(sid)[2]
    assert pool.page_table[sid, :pages].cpu().numpy().tolist() == list(hot)
    assert (pool.page_table[sid, pages:].cpu() == -1).all()
    assert torch.equal(pool.hot_page_bytes(hot).cpu(), before)
    pool.extend(sid, 16 * pages + 1)
    assert pool.page_table[sid, :pages + 1].cpu().numpy().tolist() == list(pool.info(sid)[2])
    pool.destroy_session(sid)
    assert (pool.page_table.cpu() == -1).all()
    pool.close()


def test_many_sessions_and_a_list_past_one_staging_slot(dev):
    """300 sessions evicted in one call (three launches of row clears) and
    resumed in one of 66,000 pages (two uploads); clean evictions list nothing."""
    n, pages = 300, 220
    pool = _pool(n * pages + 5, n, pages + 1)
    words = pool.hot.view(torch.int32)
    words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
    sids = [pool.create_session(16 * pages) for _ in range(n)]
    want = pool.hot_page_bytes(torch.arange(n * pages))
    pool.evict(sids)
    assert (pool.page_table.cpu() == -1).all()
    pool.hot.zero_()
    order = [int(x) for x in np.random.default_rng(1).permutation(n)]
    pool.resume(order)
    table = pool.page_table[:, :pages].long()
    assert sorted(table.cpu().reshape(-1).tolist()) == list(range(n * pages))
    assert torch.equal(pool.hot_page_bytes(table.reshape(-1)), want)
    written = pool.stats()["pages_to_cold"]
    pool.evict(sids)
    assert pool.stats()["pages_to_cold"] == written == n * pages
    assert (pool.page_table.cpu() == -1).all()
    pool.close()


def test_freed_pages_wait_for_the_freeing_stream(dev):
    """A dirty eviction on one stream, then a session created on another takes
    the freed pages and writes them: the cold copies hold the old bytes."""
    pages = 3000
    pool = _pool(pages, 2, pages)
    words = pool.hot.view(torch.int32)
    words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    sid = pool.create_session(16 * pages, stream=a)
    want = pool.hot_page_bytes(torch.arange(pages)).clone()
    torch.cuda.synchronize()
    ones = torch.ones((16 * pages, 1, 64), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    pool.evict(sid, stream=a)
    other = pool.create_session(16 * pages, stream=b)
    pool.write_tokens(other, 0, 0, ones, ones, stream=b)
    torch.cuda.synchronize()
    cold = pool.info(sid)[3]
    assert torch.equal(pool.cold.view(pages, -1)[torch.tensor(list(cold), device=dev)], want)
    assert (pool.hot.view(torch.bfloat16) == 1).all()
    pool.close()


@pytest.fixture(scope="module")
def busy(dev):
    """busy(stream): some tens of milliseconds of matrix products enqueued on the stream."""
    a = torch.zeros((8192, 8192), dtype=torch.bfloat16, device=dev)
    torch.mm(a, a)
    torch.cuda.synchronize()

    def run(stream):
        with torch.cuda.stream(stream):
            for _ in range(60):
                torch.mm(a, a)
    return run


def _mark(stream):
    ev = torch.cuda.Event()
    ev.record(stream)
    return ev


@pytest.mark.parametrize("pages", [100, 3000])    # a list in the kernel arguments, an uploaded one
def test_freed_pages_wait_for_a_delayed_eviction(dev, busy, pages):
    """The eviction's copy stands behind other work of its stream when a session created on
    a second stream takes the freed pages and writes them: the writes come after the copy."""
    pool = _pool(pages, 2, pages)
    words = pool.hot.view(torch.int32)
    words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    ones = torch.ones((16 * pages, 1, 64), dtype=torch.bfloat16, device=dev)
    torch.cuda.synchronize()
    sid = pool.create_session(16 * pages, stream=a)
    want = pool.hot_page_bytes(torch.arange(pages)).clone()
    torch.cuda.synchronize()
    busy(a)
    pool.evict(sid, stream=a)
    evicted = _mark(a)
    other = pool.create_session(16 * pages, stream=b)
    pool.write_tokens(other, 0, 0, ones, ones, stream=b)
    assert not evicted.query(), "the delay was too short for the test to show anything"
    torch.cuda.synchronize()
    cold = pool.info(sid)[3]
    assert torch.equal(pool.cold.view(pages, -1)[torch.tensor(list(cold), device=dev)], want)
    assert (pool.hot.view(torch.bfloat16) == 1).all()
    pool.close()


@pytest.mark.parametrize("sessions", [1, 300])    # one launch of row clears, three
@pytest.mark.parametrize("how", ["destroy", "evict"])
def test_new_rows_wait_for_delayed_clears(dev, busy, sessions, how):
    """Rows cleared without a copy (sessions destroyed, or evicted while their cold copies
    are valid) on a delayed stream; the sessions created, or resumed, on a second stream
    write the same rows, after the clears."""
    pages = 3
    pool = _pool(sessions * pages, sessions, pages)
    pool.hot.zero_()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    sids = [pool.create_session(16 * pages, stream=a) for _ in range(sessions)]
    pool.evict(sids, stream=a)
    pool.resume(sids, stream=a)
    torch.cuda.synchronize()
    moved = pool.stats()["pages_to_cold"]
    busy(a)
    if how == "evict":
        pool.evict(sids, stream=a)
    else:
        for s in sids:
            pool.destroy_session(s, stream=a)
    cleared = _mark(a)
    if how == "evict":
        pool.resume(sids, stream=b)
    else:
        assert sorted(pool.create_session(16 * pages, stream=b) for _ in range(sessions)) == sorted(sids)
    assert not cleared.query(), "the delay was too short for the test to show anything"
    torch.cuda.synchronize()
    assert pool.stats()["pages_to_cold"] == moved
    table = pool.page_table.cpu().numpy()
    assert all(table[s].tolist() == list(pool.info(s)[2]) for s in sids)
    assert sorted(table.reshape(-1).tolist()) == list(range(sessions * pages))
    pool.close()


def test_evictions_and_destroys_in_a_graph(dev):
    """Captured evictions (a list in the kernel arguments, an uploaded list) and a destroy:
    each replay copies the pages and clears the rows as the eager calls do."""
    lens = [5, 200, 3]
    n = sum(lens)

    def build():
        pool = _pool(n, 3, max(lens) + 1)
        words = pool.hot.view(torch.int32)
        words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
        pool.cold.zero_()
        for p in lens:
            pool.create_session(16 * p)
        torch.cuda.synchronize()
        return pool

    def work(pool, stream=None):
        pool.evict(0, stream=stream)
        pool.evict([1], stream=stream)
        pool.destroy_session(2, stream=stream)

    eager = build()
    work(eager)
    torch.cuda.synchronize()
    assert int(eager.cold.count_nonzero()) > 0 and (eager.page_table == -1).all()
    pool = build()
    table = pool.page_table.clone()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        work(pool, s)
    assert torch.equal(pool.page_table, table) and int(pool.cold.count_nonzero()) == 0
    for _ in range(3):
        pool.cold.zero_()
        pool.page_table.copy_(table)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(pool.cold, eager.cold)
        assert torch.equal(pool.page_table, eager.page_table)
    pool.close()
    eager.close()


@pytest.mark.parametrize("pages", [7, 200])
def test_eager_calls_after_a_captured_one(dev, pages):
    """The stream's mark and a staging slot's event, recorded in a capture first, are
    recorded by eager calls after it, and other streams wait for those."""
    pool = _pool(5 * pages, 5, pages + 1)
    words = pool.hot.view(torch.int32)
    words.copy_(torch.arange(words.numel(), dtype=torch.int32, device=dev))
    for _ in range(5):
        pool.create_session(16 * pages)
    want = pool.hot_page_bytes(torch.arange(5 * pages)).clone()
    torch.cuda.synchronize()
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        pool.evict(0, stream=s)
    g.replay()
    torch.cuda.synchronize()
    for stream in (s, t):
        pool.evict([1, 2], stream=s)
        pool.resume([2, 1], stream=stream)
        torch.cuda.synchronize()
    pool.evict([1, 2, 3, 4], stream=t)
    torch.cuda.synchronize()
    assert (pool.page_table == -1).all()
    for sid in range(5):
        cold = torch.tensor(list(pool.info(sid)[3]), device=dev)
        assert torch.equal(pool.cold.view(5 * pages, -1)[cold], want[sid * pages:(sid + 1) * pages])
    pool.close()
