"""The sampler's later hops through hash buckets in LDS: sizes at the edges of its tiles and of the
fanouts it keeps in registers, ids that all fall into one bucket, and a workspace without room for
buckets.  Everything is compared with the oracle element by element (tolerance zero)."""
import ctypes as C
import time

import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_sample, dev, ginex, small_graph  # noqa: F401

pytestmark = pytest.mark.gpu


def both(ginex, off, ind, batches, fanout, **kw):
    seeds = np.concatenate(batches).astype(np.int32)
    so = np.cumsum([0] + [len(b) for b in batches])
    ref = oracle.sample_superbatch(off, ind, seeds, so, fanout, rng_seed=5, first_batch_index=2)
    res = ginex.sample_superbatch(dev(off), dev(ind), dev(seeds), so, fanout, rng_seed=5,
                                  first_batch_index=2, **kw)
    check_sample(res, ref, len(batches), len(fanout))


# more than 1024 seeds: the first hop's frontier has exactly as many nodes as the batch has seeds
@pytest.mark.parametrize("k", [1, 16, 17, 32, 33])
@pytest.mark.parametrize("offsets_64", [False, True])
def test_frontiers_around_the_tile_sizes(ginex, k, offsets_64):  # noqa: F811
    off, ind = small_graph(n=6000, e=150_000, offsets_64=offsets_64)
    rng = np.random.default_rng(k)
    batches = [rng.choice(6000, size=n, replace=False) for n in (1025, 2047, 2048, 2049, 2303, 2304, 2305, 3)]
    both(ginex, off.numpy(), ind.numpy(), batches, (k, 3))


# fewer batches than XCDs are dealt to all of them, from 33 tiles of a batch on; both ways of a hop, one or
# several tiles to a block
@pytest.mark.parametrize("S", [1, 2, 3, 7, 8, 9])
@pytest.mark.parametrize("lds,tiles", [("1", "0"), ("0", "0"), ("1", "2"), ("1", "32"), ("1", "33"), ("0", "33")])
def test_numbers_of_batches_around_the_xcds(ginex, S, lds, tiles, monkeypatch):  # noqa: F811
    monkeypatch.setenv("GINEX_SAMPLER_LDS", lds)
    monkeypatch.setenv("GINEX_SAMPLER_TILES", tiles)
    off, ind = small_graph(n=6000, e=150_000)
    rng = np.random.default_rng(S)
    batches = [rng.choice(6000, size=int(rng.integers(1, 1500)), replace=False) for _ in range(S)]
    both(ginex, off.numpy(), ind.numpy(), batches, (7, 5))


def wide_graph(n, degree):
    """Every node has `degree` neighbours, drawn with repetitions."""
    off = np.arange(n + 1, dtype=np.int64) * degree
    return off, np.random.default_rng(degree).integers(0, n, off[-1]).astype(np.int32)


# 1.5 M ids in a batch: the bound on either side, the bound beyond it and the lists below, both beyond
@pytest.mark.parametrize("seeds,degree", [(12_000, 12), (12_397, 12), (13_000, 6), (13_000, 12)])
def test_batches_around_the_most_ids_of_the_buckets(ginex, seeds, degree):  # noqa: F811
    n = 3_000_000
    off, ind = wide_graph(n, degree)
    batches = [np.random.default_rng(seeds).choice(n, size=m, replace=False) for m in (5, seeds, 0)]
    both(ginex, off, ind, batches, (10, 10))


def test_large_batches_cost_no_more_than_the_tables(ginex, monkeypatch):  # noqa: F811
    """A batch far beyond what the buckets hold, against the tables in HBM, best of four (in slices it
    took nine times as long)."""
    n = 20_000_000
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * 12
    ind = torch.randint(n, (12 * n,), dtype=torch.int32, device="cuda")
    seeds, so = torch.randperm(n, device="cuda")[:4000].int(), np.array([0, 4000])
    best = {}
    for lds in ("0", "1"):
        monkeypatch.setenv("GINEX_SAMPLER_LDS", lds)
        times = []
        for _ in range(4):
            torch.cuda.synchronize()
            began = time.perf_counter()
            ginex.sample_superbatch(off, ind, seeds, so, (10, 10, 10))
            times.append(time.perf_counter() - began)
        best[lds] = min(times)
    assert best["1"] < 1.5 * best["0"], best


# empty batches have no tiles and no buckets; alone, between others, and in front of a first hop that
# goes through buckets (1025 seeds) or through one workgroup's LDS
@pytest.mark.parametrize("sizes", [(0,), (0, 0, 0), (0, 1025, 0, 7, 0, 0, 300, 0, 0), (0, 90, 0, 1)])
def test_empty_batches(ginex, sizes):  # noqa: F811
    off, ind = small_graph(n=6000, e=150_000)
    rng = np.random.default_rng(len(sizes))
    batches = [rng.choice(6000, size=n, replace=False) for n in sizes]
    both(ginex, off.numpy(), ind.numpy(), batches, (8, 3))


def fmix32(h):
    h = h.astype(np.uint32)
    h ^= h >> np.uint32(16)
    h *= np.uint32(0x85EBCA6B)
    h ^= h >> np.uint32(13)
    h *= np.uint32(0xC2B2AE35)
    return h ^ (h >> np.uint32(16))


# 6 400 ids in the first of 512 buckets, whose table has 4 096 slots: done in slices
@pytest.mark.parametrize("repeats", [False, True])
def test_ids_that_fall_into_one_bucket(ginex, repeats):  # noqa: F811
    N, seeds, mid, k = 4_000_000, 20, 10, 32
    ids = np.arange(1000, N, dtype=np.uint32)
    pool = ids[fmix32(ids) < np.uint32((1 << 32) // 512)][:seeds * mid * k].astype(np.int64)
    assert len(pool) == seeds * mid * k
    if repeats:                       # and many of them twice
        pool = pool[np.random.default_rng(1).integers(0, len(pool), len(pool))]
    deg = np.zeros(N, dtype=np.int64)
    deg[:seeds] = mid
    deg[100:100 + seeds * mid] = k
    off = np.zeros(N + 1, dtype=np.int64)
    np.cumsum(deg, out=off[1:])
    ind = np.empty(off[-1], dtype=np.int32)
    ind[:seeds * mid] = 100 + np.arange(seeds * mid)
    ind[seeds * mid:] = pool
    both(ginex, off, ind, [np.arange(seeds)], (mid, k))


def test_workspace_without_room_for_buckets(ginex):  # noqa: F811
    """On a small graph the buckets take more room than the tables: a workspace that only has room
    for the tables is still accepted, and gives the same result."""
    off, ind = small_graph()
    off, ind = off.cuda(), ind.cuda()
    seeds = dev(np.arange(200, dtype=np.int32))
    so, fo = np.array([0, 90, 200]), np.array([9, 9, 9], dtype=np.int32)
    full = ginex.sample_superbatch(off, ind, seeds, so, fo)
    lib = ginex._lib.load()
    n = off.numel() - 1
    need = lib.ginex_sample_workspace_bytes(n, 2, 110, fo.ctypes.data, 3)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    ids = torch.empty_like(full.ids)
    rowptr, col = torch.empty_like(full.adj_rowptr), torch.empty_like(full.adj_col)
    so = so.astype(np.int64)
    ids_off, hops = np.zeros(3, np.int64), np.zeros(8, np.int64)
    rows, cols, totals = np.zeros(7, np.int64), np.zeros(7, np.int64), np.zeros(3, np.int64)
    g = ginex._lib.CsrDesc(n, ind.numel(), off.data_ptr(), int(off.dtype == torch.int64),
                           ind.data_ptr(), None, None)
    p = lambda a: C.c_void_p(a.ctypes.data if isinstance(a, np.ndarray) else a.data_ptr())  # noqa: E731

    def call(nbytes):
        rc = lib.ginex_sample_superbatch(
            C.byref(g), p(seeds), p(so), 2, p(fo), 3, 0, 0, p(ids), ids.numel(), p(ids_off), p(hops),
            p(rowptr), rowptr.numel(), p(col), col.numel(), p(rows), p(cols), p(totals), p(ws), nbytes,
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
        if rc == 0:
            assert torch.equal(ids, full.ids) and torch.equal(rowptr, full.adj_rowptr)
            assert torch.equal(col, full.adj_col) and np.array_equal(hops, full.hop_sizes.ravel())
        return rc

    assert call(need) == 0
    lo, hi = 0, need                  # the smallest size that is accepted
    while lo < hi:
        mid = (lo + hi) // 2
        if call(mid) == 0:
            hi = mid
        else:
            lo = mid + 1
    assert lo < need


# fanouts k above 16 of up to 2 048 + 512 (k - 16) frontier nodes in all (bound: seeds and their picks), or
# of 20 000 where the rows are shorter than that on the mean, keep the tables
@pytest.mark.parametrize("sizes", [(640, 300), (641, 3), (1024, 1024, 1), (1024, 1023, 1023, 1024, 1023),
                                   (3000, 3000, 3000, 1000), (3000, 3000, 3000, 1001)])
@pytest.mark.parametrize("k", [16, 17, 32])
@pytest.mark.parametrize("edges", [90_000, 250_000])
def test_wide_fanouts_of_few_nodes(ginex, sizes, k, edges):  # noqa: F811
    off, ind = small_graph(n=6000, e=edges)
    rng = np.random.default_rng(k)
    both(ginex, off.numpy(), ind.numpy(), [rng.choice(6000, size=m, replace=False) for m in sizes], (1, k, k))


# the first hop in LDS: a thread per node beyond eight seeds per pick and up to fanout 16, else groups of
# 16, 32 or 64 lanes
@pytest.mark.parametrize("k", [1, 2, 5, 10, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("offsets_64", [False, True])
def test_first_hop_by_node_and_by_group(ginex, k, offsets_64):  # noqa: F811
    off, ind = small_graph(n=6000, e=150_000, offsets_64=offsets_64)
    rng = np.random.default_rng(k)
    most = min(1024, 12288 // (k + 1))
    for widest in {1, min(8 * k, most), min(8 * k + 1, most), most}:
        batches = [rng.choice(6000, size=n, replace=False) for n in (widest, 0, max(1, widest // 2))]
        both(ginex, off.numpy(), ind.numpy(), batches, (k,))


# neighbour ids behind the host link keep the group of lanes per node; with a neighbour cache in HBM in
# front of them, and with the same ids in HBM, the lists are the same
@pytest.mark.parametrize("k", [1, 16, 32])
def test_neighbour_ids_in_host_memory(ginex, k):  # noqa: F811
    off, ind = small_graph(n=6000, e=150_000)
    rng = np.random.default_rng(k)
    batches = [rng.choice(6000, size=n, replace=False) for n in (1025, 2305, 3)]
    seeds = np.concatenate(batches).astype(np.int32)
    so = np.cumsum([0] + [len(b) for b in batches])
    ref = oracle.sample_superbatch(off.numpy(), ind.numpy(), seeds, so, (k, 3), rng_seed=5,
                                   first_batch_index=2)
    pinned = torch.empty(ind.numel(), dtype=torch.int32, pin_memory=True)
    pinned.copy_(ind)
    nc = ginex.neighbor_cache_build(dev(off.numpy()), pinned, 40_000)
    for indices, cache in ((pinned, None), (pinned, nc), (ind.cuda(), nc)):
        res = ginex.sample_superbatch(dev(off.numpy()), indices, dev(seeds), so, (k, 3), rng_seed=5,
                                      first_batch_index=2, neighbor_cache=cache)
        check_sample(res, ref, len(batches), 2)
