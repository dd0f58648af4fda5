"""The split's unit stream at its edges (GPU): a wave walks consecutive pages of
many rows, 60 to 64 of them per chunk, with its ring running on from row to row."""

import numpy as np
import pytest
import torch

import synth
from helpers import Case, build_gpu, rowwise_check, to_device, to_host, tolerance_check

pytestmark = pytest.mark.gpu

# runs of empty rows, rows of one to three pages (shorter than the ring), rows
# that end on a chunk's last unit and one past it, and one of several chunks
LENS = [1, 0, 0, 0, 16, 17, 33, 48, 5, 0, 60 * 16, 1, 63 * 16, 64 * 16 + 1, 2, 18, 0, 200 * 16 - 7, 31, 32, 0, 0]


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda", 0)


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("dtype,D,hq,hkv,waves", [
    ("bf16", 128, 16, 4, 4), ("bf16", 128, 16, 4, 768), ("bf16", 64, 16, 16, 8), ("bf16", 64, 6, 2, 1),
    ("f32", 128, 8, 8, 12), ("f32", 64, 4, 1, 3)])
def test_rows_of_every_length_against_the_oracle(dev, dtype, D, hq, hkv, waves, fused):
    """One to four head groups per row and workers of one and four waves; with
    few waves each walks several chunks."""
    case = Case(1, hq, hkv, D, dtype, LENS, seed=41)
    pool = build_gpu(case, dev, poison=True)
    pool.set_waves(waves)
    pool.set_combine(fused)
    got = to_host(pool.decode(0, to_device(case.q, dtype, dev), torch.tensor(LENS, dtype=torch.int32, device=dev)))
    pool.close()
    rowwise_check(got, case.oracle_out(), max_norm=1e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("dtype,D,hq,hkv,waves", [
    ("bf16", 128, 16, 4, 4), ("bf16", 64, 16, 16, 8), ("f32", 128, 8, 8, 12), ("f32", 64, 4, 1, 3),
    ("bf16", 128, 8, 1, 64)])
def test_append_into_consecutive_short_rows(dev, dtype, D, hq, hkv, waves):
    """Tail pages one to three units apart: a wave holds one row's new token
    while it meets the next ones'.  Bitwise equal to a separate append, pages
    included."""
    kvs = [synth.session_kv(43, b, L, 0, hkv, D, 1.0, dtype) for b, L in enumerate(LENS)]
    case = Case(1, hq, hkv, D, dtype, LENS, seed=43)
    q = to_device(case.q, dtype, dev)
    sl = torch.tensor(LENS, dtype=torch.int32, device=dev)
    rows = [b for b, L in enumerate(LENS) if L]
    new = [np.zeros((len(LENS), hkv, D), kvs[0][0].dtype) for _ in range(2)]
    for b in rows:
        for i in range(2):
            new[i][b] = kvs[b][i][LENS[b] - 1]
    kn, vn = (to_device(t, dtype, dev) for t in new)
    outs, hots = [], []
    for fused_append in (True, False):
        pool = build_gpu(case, dev, poison=True)
        pool.set_waves(waves)
        for b in rows:   # the last token's slot holds NaN until it is appended
            nan = torch.full((1, hkv, D), float("nan"), dtype=kn.dtype, device=dev)
            pool.write_tokens(b, 0, LENS[b] - 1, nan, nan)
        if fused_append:
            outs.append(pool.decode(0, q, sl, k_new=kn, v_new=vn).clone())
        else:
            pool.append_tokens(0, rows, [LENS[b] - 1 for b in rows], kn[rows].contiguous(), vn[rows].contiguous())
            outs.append(pool.decode(0, q, sl).clone())
        torch.cuda.synchronize()
        hots.append(pool.hot.clone())
        pool.close()
    assert torch.equal(hots[0], hots[1])
    assert torch.equal(outs[0], outs[1])
    tolerance_check(to_host(outs[0]), case.oracle_out(), max_norm=1e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("dtype,D,group", [("bf16", 128, 8), ("bf16", 64, 3), ("f32", 128, 4), ("f32", 64, 16)])
@pytest.mark.parametrize("waves", [11, 12, 63, 64, 65, 300])
def test_merge_widths(dev, dtype, D, group, waves):
    """One row, so `waves` partials per head: one, four and sixteen waves per
    head merge them, below, at and above the rule's edges."""
    lens = [16 * 333 - 5]
    case = Case(1, group, 1, D, dtype, lens, seed=47)
    pool = build_gpu(case, dev)
    pool.set_waves(waves)
    got = to_host(pool.decode(0, to_device(case.q, dtype, dev), torch.tensor(lens, dtype=torch.int32, device=dev)))
    pool.close()
    tolerance_check(got, case.oracle_out(), max_norm=1e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("batch", [1, 62, 63, 64, 65, 255, 256, 257, 600])
def test_row_prefix_of_so_many_rows(dev, batch):
    """The prefix sum of a wave's worth of rows, of a block's worth and of more,
    empty rows among them; the partition table uses the same sum."""
    from oracle import partition
    rng = np.random.default_rng(batch)
    lens = [int(x) for x in rng.integers(0, 70, size=batch)]
    lens[-1] = 33
    case = Case(1, 4, 2, 64, "bf16", lens, seed=53)
    pool = build_gpu(case, dev)
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    got = to_host(pool.decode(0, to_device(case.q, "bf16", dev), sl))
    slots = pool.partition(sl, 24).cpu().numpy()
    pool.close()
    tolerance_check(got, case.oracle_out())
    assert np.array_equal(slots, np.array(partition.slot_table(lens, 2, 24), dtype=np.int32))


@pytest.mark.parametrize("dtype,D,hq,hkv,batch", [
    ("bf16", 128, 32, 4, 90),    # the model's shape: rows of 2 KiB per KV head
    ("bf16", 128, 16, 1, 90),    # 16 heads per group: the partial is not held
    ("bf16", 64, 16, 2, 90),     # 1 KiB exactly
    ("bf16", 64, 14, 2, 90),     # below 1 KiB: rows stored as they end
    ("f32", 128, 8, 1, 90),      # two slots
    ("f32", 128, 16, 1, 90),     # room for one slot only: rows stored as they end
    ("bf16", 128, 8, 1, 5000),   # the row prefix takes 20 KB of the LDS
])
@pytest.mark.parametrize("waves", [3, 4, 8])
def test_rows_held_until_slots_fill(dev, dtype, D, hq, hkv, batch, waves):
    """More segments than waves: each wave finishes many whole rows, more than it
    can hold at once, among them empty rows and one bad page id (a NaN row).
    The output starts as NaN: every row must be written."""
    rng = np.random.default_rng(batch + waves)
    lens = [int(x) for x in (rng.integers(1, 120, size=batch) if batch < 1000 else rng.integers(1, 18, size=batch))]
    lens[4] = lens[5] = 0
    case = Case(1, hq, hkv, D, dtype, lens, seed=59)
    pool = build_gpu(case, dev, poison=True)
    pool.set_waves(waves)
    q = to_device(case.q, dtype, dev)
    table = pool.page_table.clone()
    table[7, 0] = case.hot_pages
    out = torch.full_like(q, float("nan"))
    pool.decode(0, q, torch.tensor(lens, dtype=torch.int32, device=dev), page_table=table, out=out)
    got = to_host(out)
    pool.close()
    assert np.isnan(got[7]).all()
    assert (got[4:6] == 0).all()
    rows = [b for b in range(batch) if lens[b] and b != 7][:: max(1, batch // 300)]
    rowwise_check(got[rows], case.oracle_out(rows=rows), max_norm=1e-2 if dtype == "bf16" else 1e-5)
    assert np.isfinite(np.delete(got, 7, axis=0)).all()


# 387 lies halfway between two bfloat16 values and is the mean of 386 and 388; for these
# token counts the float32 product 387 n * (1 / n) falls below it, the quotient does not
HALFWAY_LENS = [n for n in range(2, 1024, 2)
                if np.float32(387 * n) * (np.float32(1) / np.float32(n)) < np.float32(387)]


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("group", [8, 2])          # rows held in LDS, rows stored as they end
@pytest.mark.parametrize("waves", [4, 768])        # whole rows and merged partials
def test_bf16_outputs_are_rounded_quotients(dev, group, waves, fused):
    """Zero queries make every weight 1, so each output is a sum of small integers over
    the token count, both exact in float32: 387, which rounds to even, 388.  A result one
    float32 unit below 387 rounds to 386."""
    from paper_2609_25782_amd.pool import HotColdPool
    lens, D = HALFWAY_LENS, 64
    assert len(lens) > 20
    pages = [synth.pages_for(L) for L in lens]
    pool = HotColdPool(1, 1, D, "bf16", sum(pages), 0, len(lens), max(pages))
    for L in lens:
        k = torch.zeros((L, 1, D), dtype=torch.bfloat16, device=dev)
        v = torch.full_like(k, 386)
        v[1::2] = 388
        pool.write_tokens(pool.create_session(L), 0, 0, k, v)
    pool.set_waves(waves)
    pool.set_combine(fused)
    q = torch.zeros((len(lens), group, D), dtype=torch.bfloat16, device=dev)
    got = to_host(pool.decode(0, q, torch.tensor(lens, dtype=torch.int32, device=dev)))
    pool.close()
    assert (got == 388).all(), np.unique(got, return_counts=True)


@pytest.mark.parametrize("tiered", [False, True])
def test_fused_append_keeps_pages_in_flight(dev, tiered):
    """A row's new token costs something at its last page and nothing at the others: on
    rows of 8K tokens the split with the append takes at most 1.3 times the one without
    (measured 1.02 to 1.08; a wait for the pages in flight at every page makes it 1.8)."""
    from paper_2609_25782_amd import hotcold_kv as kv
    from paper_2609_25782_amd.pool import HotColdPool
    B, L, heads, D = 24, 8192, 16, 64
    pages = B * L // 16
    cold = pages // 3 if tiered else 0
    pool = HotColdPool(1, heads, D, "bf16", pages - cold, cold, B, L // 16)
    pool.set_spill(tiered)
    pool.hot.zero_()
    pool.cold.zero_()
    for _ in range(B):
        pool.create_session(L)
    q = torch.ones((B, heads, D), dtype=torch.bfloat16, device=dev)
    lens = torch.full((B,), L, dtype=torch.int32, device=dev)

    def split_ms(**new):
        for _ in range(5):
            pool.decode(0, q, lens, **new)
        torch.cuda.synchronize()
        kv.kv_pool_set_profiling(pool.handle, True)
        for _ in range(30):
            pool.decode(0, q, lens, **new)
        torch.cuda.synchronize()
        calls, ms = kv.kv_pool_profile_read(pool.handle, kv.KV_KERNEL_DECODE_SPLIT)
        kv.kv_pool_set_profiling(pool.handle, False)
        return ms / calls
    plain, append = split_ms(), split_ms(k_new=q, v_new=q)
    pool.close()
    assert append < 1.3 * plain, (plain, append)


@pytest.mark.parametrize("dtype,D,group", [
    ("bf16", 64, 4), ("bf16", 64, 5), ("bf16", 128, 4), ("bf16", 128, 5), ("bf16", 128, 16), ("f32", 64, 16),
    ("f32", 128, 1), ("f32", 128, 9)])
@pytest.mark.parametrize("waves", [3, 17, 300, 1000])
def test_fused_merge_of_every_width(dev, dtype, D, group, waves):
    """Groups whose (head, 4-dim quad) items are 64, 128, 256 and more, so that the merging
    wave takes 16, 8 and 4 partials at a time, of one row cut into fewer and more pieces
    (one per page with more waves than pages), beside a whole short row."""
    lens = [16 * 333 - 5, 7]
    case = Case(1, group, 1, D, dtype, lens, seed=67)
    pool = build_gpu(case, dev)
    pool.set_waves(waves)
    pool.set_combine(True)
    q, sl = to_device(case.q, dtype, dev), torch.tensor(lens, dtype=torch.int32, device=dev)
    outs = [to_host(pool.decode(0, q, sl)) for _ in range(3)]    # counters back at zero after each
    pool.close()
    rowwise_check(outs[0], case.oracle_out(), max_norm=1e-2 if dtype == "bf16" else 1e-5)
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("dtype,D,pages", [
    (dtype, D, n) for dtype, D in (("bf16", 128), ("f32", 64)) for n in (1, 7, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 200)])
def test_merge_is_the_same_for_every_table_stride(dev, dtype, D, pages):
    """A row's partials are at most its table row's entries, and the merge takes no more
    waves than those give work to: the same result, bit for bit, through a table that is
    just wide enough and through a wide one."""
    lens = [16 * pages - 3]
    case = Case(1, 2, 1, D, dtype, lens, seed=71, extra_stride=0)
    pool = build_gpu(case, dev)
    q, sl = to_device(case.q, dtype, dev), torch.tensor(lens, dtype=torch.int32, device=dev)
    outs = []
    for stride in (pages, 16 * pages + 4000):
        table = torch.full((1, stride), -1, dtype=torch.int32, device=dev)
        table[:, :pages] = pool.page_table
        outs.append(pool.decode(0, q, sl, page_table=table).clone())
    pool.close()
    assert torch.equal(outs[0], outs[1])
    tolerance_check(to_host(outs[0]), case.oracle_out(), max_norm=1e-2 if dtype == "bf16" else 1e-5)


def test_fused_append_waits_for_no_page_but_its_own(dev):
    """Spilled ragged rows of 8K to 32K tokens, 16 KV heads: the split with the append takes
    at most 1.05 times the one without (measured 1.02; 1.09 when every tail page, and each
    round of the ring, waited for the pages in flight).  Best of six turns on each side."""
    from paper_2609_25782_amd import hotcold_kv as kv
    from paper_2609_25782_amd.pool import HotColdPool
    heads, D = 16, 64
    lens = [int(x) for x in np.random.default_rng(5).integers(8192, 32769, size=32)]
    pages = sum(synth.pages_for(L) for L in lens)
    cold = int(0.4 * pages)
    pool = HotColdPool(1, heads, D, "bf16", pages - cold + 4, cold + 4, len(lens), max(lens) // 16 + 1)
    pool.set_spill(True)
    pool.hot.zero_()
    pool.cold.zero_()
    for L in lens:
        pool.create_session(L)
    q = torch.ones((len(lens), heads, D), dtype=torch.bfloat16, device=dev)
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)

    def split_ms(**new):
        kv.kv_pool_set_profiling(pool.handle, True)
        for _ in range(10):
            pool.decode(0, q, sl, **new)
        torch.cuda.synchronize()
        calls, ms = kv.kv_pool_profile_read(pool.handle, kv.KV_KERNEL_DECODE_SPLIT)
        kv.kv_pool_set_profiling(pool.handle, False)
        return ms / calls
    turns = [(split_ms(), split_ms(k_new=q, v_new=q)) for _ in range(7)][1:]
    pool.close()
    plain, append = min(t[0] for t in turns), min(t[1] for t in turns)
    assert append < 1.05 * plain, (plain, append)


@pytest.mark.parametrize("dtype,D,hq,hkv", [
    ("bf16", 128, 32, 4), ("bf16", 64, 16, 2), ("f32", 128, 8, 1), ("f32", 64, 8, 2)])
@pytest.mark.parametrize("waves", [3, 4, 8])
@pytest.mark.parametrize("append", [False, True])
def test_rows_held_of_hot_and_spilled_pages(dev, dtype, D, hq, hkv, waves, append):
    """Held rows over both tiers: every third row spilled, some of its pages promoted again,
    so that a wave's chunk goes from hot pages to spilled ones and back, between rows and
    inside one.  Against the oracle, and with the append bit for bit against a separate
    append, the pages of both tiers included."""
    rng = np.random.default_rng(10 * waves + D)
    lens = [int(x) for x in rng.integers(1, 120, size=90)]
    lens[4] = lens[5] = 0
    lens[30] = 16 * 70 - 3    # a spilled row longer than a chunk
    case = Case(1, hq, hkv, D, dtype, lens, seed=73)
    q, sl = to_device(case.q, dtype, dev), torch.tensor(lens, dtype=torch.int32, device=dev)
    rows = [b for b, L in enumerate(lens) if L]
    new = [np.zeros((len(lens), hkv, D), case.kv[0][0].dtype) for _ in range(2)]
    for b in rows:
        for i in range(2):
            new[i][b] = case.kv[b][i][lens[b] - 1]
    kn, vn = (to_device(t, dtype, dev) for t in new)
    nan = torch.full((1, hkv, D), float("nan"), dtype=kn.dtype, device=dev)
    outs, pages = [], []
    for form in ("fused", "separate") if append else ("plain",):
        pool = build_gpu(case, dev, num_cold_pages=case.hot_pages, poison=True)
        pool.cold.zero_()
        pool.set_waves(waves)
        pool.set_spill(True)
        if append:    # the last token's slot holds NaN until it is appended
            for b in rows:
                pool.write_tokens(b, 0, lens[b] - 1, nan, nan)
        spilled = [b for b in rows if b % 3 == 0]
        pool.evict(spilled)
        pool.resume_lazy(spilled)
        assert pool.promote(sum(synth.pages_for(lens[b]) for b in spilled) // 2 + 1) > 0
        tier = (pool.page_table >> 29).cpu().numpy()
        mixed = [b for b in rows if len(set(tier[b, :synth.pages_for(lens[b])])) > 1]
        assert mixed and (tier == 2).any() and (tier == 0).any()
        out = torch.full_like(q, float("nan"))
        if form == "fused":
            pool.decode(0, q, sl, out=out, k_new=kn, v_new=vn)
        else:
            if form == "separate":
                pool.append_tokens(0, rows, [lens[b] - 1 for b in rows], kn[rows].contiguous(), vn[rows].contiguous())
            pool.decode(0, q, sl, out=out)
        torch.cuda.synchronize()
        outs.append(out)
        pages.append((pool.hot.clone(), pool.cold.clone()))
        pool.close()
    got = to_host(outs[0])
    assert (got[4:6] == 0).all()
    rowwise_check(got[rows], case.oracle_out(rows=rows), max_norm=1e-2 if dtype == "bf16" else 1e-5)
    if append:
        assert torch.equal(outs[0], outs[1])
        assert torch.equal(pages[0][0], pages[1][0]) and torch.equal(pages[0][1], pages[1][1])
