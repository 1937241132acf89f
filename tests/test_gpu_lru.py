"""LRU changesets from the trace alone against the loop over the cache state and the oracle (tolerance zero):
caches around the longest iteration (below it only the loop serves), numbers of iterations around the
waves and blocks of the kernels, rows accessed in every iteration, empty iterations."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu


def trace(rng, n, lengths, hot):
    """Distinct ids per iteration: `hot` ids come in every one of them that is long enough."""
    parts = []
    for k in lengths:
        first = rng.permutation(hot)[:k]
        rest = rng.choice(np.arange(hot, n), size=k - len(first), replace=False)
        parts.append(rng.permutation(np.concatenate([first, rest])))
    return np.concatenate(parts).astype(np.int32), np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


@pytest.mark.parametrize("S,longest,hot", [(1, 3000, 5), (2, 3000, 900), (7, 700, 300), (20, 2500, 0), (63, 300, 40),
                                           (64, 300, 40), (65, 300, 299), (256, 90, 3), (1024, 40, 7), (1025, 40, 7),
                                           (2047, 30, 2), (2048, 30, 2), (2049, 30, 2)])
def test_caches_around_the_longest_iteration(ginex, S, longest, hot, monkeypatch):  # noqa: F811
    rng = np.random.default_rng(S)
    lengths = rng.integers(longest // 2, longest + 1, S)
    lengths[rng.integers(0, S)] = longest
    if S > 3:
        lengths[rng.integers(0, S, 2)] = 0
    n = 6 * longest
    ids, off = trace(rng, n, lengths, hot)
    distinct, most = len(np.unique(ids)), int(lengths.max())
    for cap in sorted({most - 1, most, most + 1, (most + distinct) // 2, distinct - 1}):
        ref = oracle.changeset_lru(n, ids, off, cap)
        for way in ("1", "0"):
            monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", way)
            check_changeset(ginex.changeset(n, dev(ids), off, cap, policy="lru"), ref, (n, ids, off))
        monkeypatch.delenv("GINEX_STATIC_THRESHOLDS")
        check_changeset(ginex.changeset(n, dev(ids), off, cap, policy="lru"), ref, (n, ids, off))


# few large iterations, where blocks of lines and tiles have many entries; sizes beyond the oracle's reach
@pytest.mark.parametrize("n,S,length,cap", [(4_000_000, 12, 400_000, 1_000_000), (9_000_000, 6, 2_500_000, 4_500_000),
                                            (9_000_000, 6, 2_500_000, 2_500_000), (60_000_000, 40, 30_000, 31_000),
                                            # few changes, few of many lines; counters of 2^24 lines fit LDS, of more not
                                            (3_000_000, 40, 60_000, 1_000_000), (20_000_000, 12, 600_000, 4_000_000),
                                            (40_000_000, 5, 8_000_000, 2**24), (40_000_000, 5, 8_000_000, 2**24 + 1)])
def test_large_traces_equal_the_loop(ginex, n, S, length, cap, monkeypatch):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(cap)
    off = np.arange(S + 1, dtype=np.int64) * length
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:length].int() for _ in range(S)])
    results = []
    for way in ("0", "1"):
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", way)
        results.append(ginex.changeset(n, ids, off, cap, policy="lru"))
    want, got = results
    assert np.array_equal(want.miss_count, got.miss_count) and want.miss_count.sum() > 0
    assert np.array_equal(want.cs_offsets, got.cs_offsets)
    for name in ("init_ids", "in_ids", "out_ids", "in_positions", "src_line"):
        assert torch.equal(getattr(want, name), getattr(got, name)), name


# selects among more than 131 072 accesses by many blocks, for up to 85 iterations; the limit in the iteration itself
# and in earlier ones, all rows of one, ids of up to 31 bits; tiles of insertions with nearly every position
@pytest.mark.parametrize("S,n", [(3, 150_000), (85, 150_000), (86, 150_000), (3, 2_000_000_000)])
def test_limits_in_long_iterations(ginex, S, n, monkeypatch):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(S)
    lengths = [131_073 if i % 3 == 0 else 131_072 if i % 3 == 1 else 145_000 for i in range(S)]
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    pool = torch.randperm(150_000, generator=gen, device="cuda") * (n // 150_000) + (n // 150_000 - 1)
    ids = torch.cat([pool[torch.randperm(len(pool), generator=gen, device="cuda")[:k]].int() for k in lengths])
    distinct = int(torch.unique(ids).numel())
    for cap in (max(lengths), max(lengths) + 1, 148_000, distinct - 1):
        results = []
        for way in ("0", "1"):
            monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", way)
            results.append(ginex.changeset(n, ids, off, cap, policy="lru"))
        want, got = results
        assert np.array_equal(want.miss_count, got.miss_count) and want.miss_count.sum() > 0
        assert np.array_equal(want.cs_offsets, got.cs_offsets)
        for name in ("init_ids", "in_ids", "out_ids", "in_positions", "src_line"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name
