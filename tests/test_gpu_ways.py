"""Which way a changeset call takes (GINEX_TRACE=1 says so), and that the results are the oracle's on each."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu


def way(call, monkeypatch, capfd):
    """What the call returns, and what it says about its way."""
    monkeypatch.setenv("GINEX_TRACE", "1")
    capfd.readouterr()
    result = call()
    said = capfd.readouterr().err
    monkeypatch.delenv("GINEX_TRACE")
    return result, said


@pytest.mark.parametrize("env,policy,cap,expected", [
    ({}, "belady", 1000, "every row fits, no sort"), ({}, "lru", 1000, "every row fits, no sort"),
    ({"GINEX_VALIDATE": "1"}, "belady", 1000, "every row fits, from the sorted accesses"),
    ({}, "belady", 100, "one workgroup"), ({"GINEX_VALIDATE": "1"}, "belady", 100, "one workgroup"),
    ({"GINEX_STATIC_THRESHOLDS": "1"}, "belady", 100, "from the trace"),
    ({"GINEX_STATIC_THRESHOLDS": "0"}, "belady", 100, "loop"),
    ({}, "lru", 400, "from the trace"), ({}, "lru", 299, "loop"), ({"GINEX_STATIC_THRESHOLDS": "0"}, "lru", 400, "loop"),
    ({}, "belady", 0, "no cache"), ({}, "lru", 0, "no cache")])
def test_ways_of_fresh_caches(ginex, env, policy, cap, expected, monkeypatch, capfd):  # noqa: F811
    rng = np.random.default_rng(3)
    n, S, length = 1000, 8, 300
    off = np.arange(S + 1, dtype=np.int64) * length
    ids = np.concatenate([rng.choice(n, length, replace=False) for _ in range(S)]).astype(np.int32)
    for name, value in env.items():
        monkeypatch.setenv(name, value)
    got, said = way(lambda: ginex.changeset(n, dev(ids), off, cap, policy=policy), monkeypatch, capfd)
    assert said.strip().endswith(": " + expected), said
    check_changeset(got, (oracle.changeset_lru if policy == "lru" else oracle.changeset)(n, ids, off, cap), (n, ids, off))


def test_nothing_accessed(ginex, monkeypatch, capfd):  # noqa: F811
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    got, said = way(lambda: ginex.changeset(10, none, np.zeros(4, dtype=np.int64), 5), monkeypatch, capfd)
    assert "nothing is accessed" in said and got.miss_count.sum() == 0


def crowd(n, S, spread, near, order="mixed"):
    """S iterations: `spread` ids from all of n, and near[i % len(near)] of the ids from n // 3 on."""
    gen = torch.Generator(device="cuda").manual_seed(S)
    first, parts = n // 3, []
    for i in range(S):
        far = (torch.arange(spread, device="cuda") * (n // spread) + 7919 * i) % n
        far = far[(far < first) | (far >= first + 65_536)]
        k = near[i % len(near)]
        ids = torch.cat([far, first + torch.randperm(65_536, generator=gen, device="cuda")[:k] if k else far[:0]]).int()
        parts.append(ids.sort()[0] if order == "sorted" else ids[torch.randperm(len(ids), generator=gen, device="cuda")])
    return torch.cat(parts), np.concatenate([[0], np.cumsum([len(x) for x in parts])]).astype(np.int64)


NO_SORT, SORTED = "every row fits, no sort", "every row fits, from the sorted accesses"


# a workgroup takes a bucket: not where one has too many ids, found by a sample of the accesses or, for few
# buckets, from the sizes; calls that are too small for that; up to ten slices of a bucket's rows
@pytest.mark.parametrize("n,S,spread,near,expected", [
    (20_000_000, 40, 20_000, (0,), NO_SORT), (20_000_000, 40, 20_000, (15_000,), SORTED),
    (20_000_000, 40, 20_000, (0, 0, 0, 9000, 0, 0, 0, 0), NO_SORT),        # two slices
    (100_000_000, 20, 60_000, (60_000,), SORTED), (100_000_000, 3, 60_000, (60_000, 0, 0), SORTED),
    (100_000_000, 2, 6000, (10_000, 0), NO_SORT),                          # 22 000 accesses are not sampled
    (100_000_000, 130, 280_000, (65_536,) + (0,) * 129, NO_SORT),          # ten slices of a whole bucket
    (100_000_000, 65, 560_000, (65_536,), SORTED),
    (3000, 300, 1000, (0,), SORTED), (3000, 30, 1000, (0,), NO_SORT)])
@pytest.mark.parametrize("order", ["mixed", "sorted"])
def test_ids_that_crowd(ginex, n, S, spread, near, expected, order, monkeypatch, capfd):  # noqa: F811
    ids, off = crowd(n, S, spread, near, order)
    cap = min(n, int(off[-1]))
    got, said = way(lambda: ginex.changeset(n, ids, off, cap), monkeypatch, capfd)
    assert said.strip().endswith(": " + expected), said
    monkeypatch.setenv("GINEX_VALIDATE", "1")
    want, said = way(lambda: ginex.changeset(n, ids, off, cap), monkeypatch, capfd)
    assert said.strip().endswith(": " + SORTED), said
    for name in ("init_ids", "src_line"):
        assert torch.equal(getattr(want, name), getattr(got, name)), name
    assert np.array_equal(want.init_ready, got.init_ready) and got.miss_count.sum() == 0


# the lines of a carried cache, the same way (from 2^21 rows on)
@pytest.mark.parametrize("n,S,spread,near,by_bucket", [
    (20_000_000, 60, 60_000, (0,), True), (20_000_000, 60, 60_000, (9000,) * 2 + (0,) * 58, True),
    (20_000_000, 60, 60_000, (15_000,), False), (16_000_000, 34, 60_000, (0,), False), (16_000_000, 36, 60_000, (0,), True)])
def test_lines_of_ids_that_crowd(ginex, n, S, spread, near, by_bucket, monkeypatch, capfd):  # noqa: F811
    ids, off = crowd(n, S, spread, near)
    rows = torch.unique(ids)
    rest = torch.arange(0, n, 11, device="cuda", dtype=torch.int32)
    start = torch.unique(torch.cat([rows[::2], rest]))
    start = torch.cat([start, rows[1::2]]).unique() if len(start) < len(rows) else start
    gen = torch.Generator(device="cuda").manual_seed(n)
    start = start[torch.randperm(len(start), generator=gen, device="cuda")]
    want = None
    for planned in ("1", "0"):
        monkeypatch.setenv("GINEX_PLANNED", planned)
        got, said = way(lambda: ginex.changeset_resume(n, ids, off, start), monkeypatch, capfd)
        if planned == "1":
            assert "planned path" in said or "stepped path" in said, said
            assert ("lines by bucket" in said) == by_bucket, said
        want = want or got
        for name in ("in_ids", "out_ids", "in_positions", "src_line", "final_ids"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name


# three lines to four accesses and more, but not certain: the rows are estimated
@pytest.mark.parametrize("n,S,length", [(10_000_000, 20, 60_000), (60_000_000, 40, 100_000), (50_000_000, 4, 2_000_001)])
def test_caches_that_may_hold_every_row(ginex, n, S, length, monkeypatch, capfd):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(n)
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:length].int() for _ in range(S)])
    off = np.arange(S + 1, dtype=np.int64) * length
    rows = int(torch.unique(ids).numel())
    assert rows * 96 // 100 * 4 >= 3 * len(ids)
    for cap, fits, tried in ((rows, True, True), (rows - 1, False, True), (rows * 97 // 100, False, False)):
        monkeypatch.delenv("GINEX_VALIDATE", raising=False)
        got, said = way(lambda: ginex.changeset(n, ids, off, cap), monkeypatch, capfd)
        assert ("no sort" in said) == fits and ("too many rows" in said) == (tried and not fits), said
        monkeypatch.setenv("GINEX_VALIDATE", "1")
        want = ginex.changeset(n, ids, off, cap)
        assert np.array_equal(want.miss_count, got.miss_count) and np.array_equal(want.cs_offsets, got.cs_offsets)
        assert np.array_equal(want.init_ready, got.init_ready)
        for name in ("init_ids", "in_ids", "out_ids", "in_positions", "src_line"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name


# LRU with just the lines that an iteration accesses: from 2^22 lines on the loop
@pytest.mark.parametrize("length,lines,expected", [(2**22, 2**22, "loop"), (2**22, 2**22 + 1, "from the trace"),
                                                   (2**22 - 1, 2**22 - 1, "from the trace")])
def test_lru_of_an_iterations_lines(ginex, length, lines, expected, monkeypatch, capfd):  # noqa: F811
    n, S = 12_000_000, 3
    gen = torch.Generator(device="cuda").manual_seed(lines)
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:length].int() for _ in range(S)])
    off = np.arange(S + 1, dtype=np.int64) * length
    got, said = way(lambda: ginex.changeset(n, ids, off, lines, policy="lru"), monkeypatch, capfd)
    assert said.strip().endswith(": " + expected), said
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1" if expected == "loop" else "0")
    want = ginex.changeset(n, ids, off, lines, policy="lru")
    assert np.array_equal(want.miss_count, got.miss_count) and np.array_equal(want.cs_offsets, got.cs_offsets)
    for name in ("init_ids", "in_ids", "out_ids", "in_positions", "src_line"):
        assert torch.equal(getattr(want, name), getattr(got, name)), name
