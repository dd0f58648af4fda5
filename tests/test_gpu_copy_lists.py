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
