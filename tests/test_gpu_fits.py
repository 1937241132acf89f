"""Fresh caches that hold every row, without a sort, against the way through the sorted accesses (which the
validating mode takes) and the oracle (tolerance zero): tiles, buckets and slices around their sizes, caches
with just enough lines and one too few."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu


def same(ginex, n, ids, off, cap, monkeypatch):  # noqa: F811
    monkeypatch.setenv("GINEX_VALIDATE", "1")
    want = ginex.changeset(n, ids, off, cap)
    monkeypatch.delenv("GINEX_VALIDATE")
    for policy in ("belady", "lru"):
        got = ginex.changeset(n, ids, off, cap, policy=policy)
        if policy == "lru" and want.miss_count.any():   # (they differ then)
            continue
        for name in ("init_ids", "in_ids", "out_ids", "in_positions", "src_line"):
            assert torch.equal(getattr(want, name), getattr(got, name)), (policy, name)
        for name in ("cs_offsets", "miss_count", "init_ready"):
            assert np.array_equal(getattr(want, name), getattr(got, name)), (policy, name)
    got = ginex.changeset(n, ids, off, cap, with_lines=False)
    assert torch.equal(want.init_ids, got.init_ids) and np.array_equal(want.init_ready, got.init_ready)
    return want


def trace(n, lengths, seed, low=None):
    """Distinct ids per iteration; low: the first ids of the graph only."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    parts = [torch.randperm(low or n, generator=gen, device="cuda")[:k].int() for k in lengths]
    return torch.cat(parts), np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


# tiles of 8 192 accesses: full, one more or less, empty iterations in between
@pytest.mark.parametrize("lengths", [(8192,) * 40, (8191, 8193) * 20, (0, 16384, 1, 0) * 24, (300_000,), (5000,) * 130])
@pytest.mark.parametrize("n", [524_288, 524_289, 3_000_017])
def test_lengths_of_iterations(ginex, n, lengths, monkeypatch):  # noqa: F811
    ids, off = trace(n, lengths, n)
    same(ginex, n, ids, off, n, monkeypatch)


@pytest.mark.parametrize("n,lengths", [(1, (1, 1)), (5, (3, 0, 5)), (2047, (300, 2047) * 2), (2048, (1, 0, 2048)),
                                       (2049, (2049, 700)), (40_000, (1,) * 300)])
def test_smallest_calls(ginex, n, lengths, monkeypatch):  # noqa: F811
    ids, off = trace(n, lengths, n)
    same(ginex, n, ids, off, n, monkeypatch)


# 2^11 to 2^16 ids to a bucket, 2 048 and 4 096 buckets, more nodes than buckets serve; the last bucket short
@pytest.mark.parametrize("n", [131_072, 4_194_304, 4_194_305, 30_000_001, 134_217_729, 268_435_456, 268_435_457])
def test_numbers_of_buckets(ginex, n, monkeypatch):  # noqa: F811
    ids, off = trace(n, (60_000, min(200_001, n - 3), 1) * 9, n)
    ids[-1] = n - 1
    ids[7] = ids[7] if bool((ids[:60_000] == n - 1).any()) else n - 1
    same(ginex, n, ids, off, ids.numel(), monkeypatch)


# a bucket's ids in a tile: 8 lanes take 8 at once, then 8 more, four times 8 up to 128, a wave the rest; ids in order (a
# bucket's lie side by side, lanes count together) and not; 128 tiles and more
@pytest.mark.parametrize("S", [11, 128, 129])
@pytest.mark.parametrize("order", ["mixed", "sorted"])
def test_shares_of_any_length(ginex, S, order, monkeypatch):  # noqa: F811
    n, bucket = 1 << 26, 1 << 15
    gen = torch.Generator(device="cuda").manual_seed(S)
    parts = []
    for i in range(S):
        k = (0, 8, 9, 16, 17, 127, 128, 129, 384, 385, 1500, 5000)[i * 7 % 12]
        near = 5 * bucket + torch.randperm(bucket, generator=gen, device="cuda")[:k]
        far = 6 * bucket + (torch.arange(3000 if k < 5000 else 3192, device="cuda") * 20011 + i * 7919) % (n - 6 * bucket)
        ids = torch.cat([near, far]).int()
        parts.append(ids.sort()[0] if order == "sorted" else ids[torch.randperm(len(ids), generator=gen, device="cuda")])
    off = np.concatenate([[0], np.cumsum([len(x) for x in parts])]).astype(np.int64)
    same(ginex, n, torch.cat(parts), off, int(off[-1]), monkeypatch)


# 7 168 rows of a bucket in LDS: all rows among the first ids, up to ten slices in a bucket and thousands of
# its ids in a tile
@pytest.mark.parametrize("low", [7168, 7169, 65_536, 65_537, 200_000])
def test_rows_in_few_buckets(ginex, low, monkeypatch):  # noqa: F811
    ids, off = trace(100_000_000, (min(low, 50_000),) * 60, low, low)
    same(ginex, 100_000_000, ids, off, ids.numel(), monkeypatch)


@pytest.mark.parametrize("S,length", [(20, 50_000), (1800, 400), (1900, 400), (3, 400_000)])
def test_caches_around_the_rows(ginex, S, length, monkeypatch):  # noqa: F811
    ids, off = trace(1 << 20, (length,) * S, S)
    rows = int(torch.unique(ids).numel())
    for cap in (rows - 1, rows, rows + 1, (ids.numel() + 1) // 2, 1 << 20):
        want = same(ginex, 1 << 20, ids, off, cap, monkeypatch)
        assert len(want.init_ids) == min(rows, cap)
    ref = oracle.changeset(1 << 20, ids.cpu().numpy(), off, rows)
    check_changeset(ginex.changeset(1 << 20, ids, off, rows), ref, (1 << 20, ids.cpu().numpy(), off))


def test_ids_out_of_range_go_the_other_way(ginex):  # noqa: F811
    """More distinct ids than nodes are refused, wherever the ids lie."""
    ids = torch.arange(90, 190, dtype=torch.int32, device="cuda")
    with pytest.raises(ginex.GinexError, match="out of range"):
        ginex.changeset(64, ids, np.array([0, 50, 100]), 64)


# fewer distinct ids than nodes, so that their number says nothing: beyond the last node in its word of the bitmap, its
# bucket, the last bucket, negative
@pytest.mark.parametrize("bad", [1000, 1023, 1024, 2047, 2048, 2**31 - 1, -1])
def test_ids_out_of_range_are_refused(ginex, bad):  # noqa: F811
    ids, off = trace(1000, (100, 0, 200), 7)
    for policy in ("belady", "lru"):
        ginex.changeset(1000, ids, off, 1000, policy=policy)
    ids[150] = bad
    for policy in ("belady", "lru"):
        for with_lines in (True, False):
            with pytest.raises(ginex.GinexError, match="out of range"):
                ginex.changeset(1000, ids, off, 1000, policy=policy, with_lines=with_lines)


# a carried cache that holds every row: its lines by bucket, up to three slices to one, rows that are not inserted;
# against the way that takes it as any other cache
@pytest.mark.parametrize("n,low,length,cap", [(20_000_000, 200_000, 150_000, 400_000), (20_000_000, 9000, 9000, 12_000),
                                              (3_000_017, 3_000_017, 80_000, 2_500_000)])
def test_lines_of_a_carried_cache(ginex, n, low, length, cap, monkeypatch):  # noqa: F811
    ids, off = trace(n, (length, 0, length - 1) * max(9, (n // 8 + (1 << 20)) // (3 * length) + 1), n, low)
    gen = torch.Generator(device="cuda").manual_seed(cap)
    start = torch.cat([torch.randperm(low, generator=gen, device="cuda")[:cap // 3],
                       n - 1 - torch.arange(cap, device="cuda")]).int().unique()
    start = start[torch.randperm(start.numel(), generator=gen, device="cuda")][:max(cap, int(ids.unique().numel()))]
    want = None
    for planned in ("0", "1"):
        monkeypatch.setenv("GINEX_PLANNED", planned)
        got = ginex.changeset_resume(n, ids, off, start)
        want = want or got
        for name in ("in_ids", "out_ids", "in_positions", "src_line", "final_ids"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name
    assert (want.src_line < 0).any() and want.cs_offsets[-1] > 0
