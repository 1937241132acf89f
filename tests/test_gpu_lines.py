"""Lines of inserted rows by blocks that wait for each other, against a launch per iteration, the loop over the cache
state and the oracle (tolerance zero): caches around the lines of a block and around what its LDS holds, iterations that
change more lines than a block hands over at a time or access more rows than it looks up at a time, waits
that are given up."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, check_resumed, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu

TOGETHER, LAUNCHES, GIVEN_UP = "all iterations together", "a launch per iteration", "given up, a launch per iteration"


def found(call, monkeypatch, capfd):
    """What the call returns, and the ways in which it says the lines were found."""
    monkeypatch.setenv("GINEX_TRACE", "2")
    capfd.readouterr()
    result = call()
    said = capfd.readouterr().err
    monkeypatch.delenv("GINEX_TRACE")
    return result, [line.split(": lines: ")[1] for line in said.splitlines() if ": lines: " in line]


NAMES = ("in_ids", "out_ids", "in_positions", "src_line", "final_ids")


def same(a, b):
    assert np.array_equal(a.miss_count, b.miss_count) and np.array_equal(a.cs_offsets, b.cs_offsets)
    for name in NAMES:
        x, y = getattr(a, name), getattr(b, name)
        assert (x is None) == (y is None) and (x is None or torch.equal(x, y)), name


# one line, around a block's 512, two blocks and a half
@pytest.mark.parametrize("policy", ["belady", "lru"])
@pytest.mark.parametrize("cap", [1, 2, 511, 512, 513, 1280])
def test_small_caches_equal_the_oracle(ginex, policy, cap, monkeypatch):  # noqa: F811
    rng = np.random.default_rng(cap)
    S, n = 11, 4 * cap + 40
    lengths = rng.integers(0, cap + 1, S)
    lengths[3], lengths[7] = cap, 0
    parts = [rng.permutation(n)[:k] for k in lengths]
    parts[5] = parts[4][::-1].copy()        # every row again in the iteration behind
    ids = np.concatenate(parts).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
    for polls in (None, "1", "0"):
        if polls:
            monkeypatch.setenv("GINEX_MOVE_POLLS", polls)
        ref = (oracle.changeset if policy == "belady" else oracle.changeset_lru)(n, ids, off, cap)
        check_changeset(ginex.changeset(n, dev(ids), off, cap, policy=policy), ref, (n, ids, off))


# the lines up to which a thread has 1, 3, 9, 17 and 35 words of LDS, and one block's more, of which the last goes back
# to a launch per iteration, LRU's behind 9 words; iterations of up to 1.2 M accesses are looked up in one go, longer ones
# in several
@pytest.mark.parametrize("cap,length", [(2**19, 400_000), (2**19 + 2, 400_000), (3 * 2**19 + 2, 700_000),
                                        (9 * 2**19, 3_000_000), (9 * 2**19 + 2, 3_000_000), (17 * 2**19 + 2, 4_000_000),
                                        (35 * 2**19, 6_000_000), (35 * 2**19 + 1, 6_000_000)])
def test_large_caches_equal_a_launch_per_iteration(ginex, cap, length, monkeypatch, capfd):  # noqa: F811
    S, n = 7, 2 * cap
    gen = torch.Generator(device="cuda").manual_seed(cap)
    off = np.arange(S + 1, dtype=np.int64) * length
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:length].int() for _ in range(S)])
    ids[4 * length:5 * length] = ids[3 * length:4 * length].flip(0)   # every row again in the iteration behind
    start = torch.randperm(n, generator=gen, device="cuda")[:cap].int()
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
    monkeypatch.setenv("GINEX_PLANNED", "0")
    for most, run in ((35, lambda lines=True: ginex.changeset(n, ids, off, cap, with_lines=lines)),
                      (9, lambda lines=True: ginex.changeset(n, ids, off, cap, policy="lru", with_lines=lines)),
                      (35, lambda lines=True: ginex.changeset_resume(n, ids, off, start, with_lines=lines))):
        monkeypatch.setenv("GINEX_MOVE_POLLS", "0")
        want, bare = run(), run(False)
        assert want.cs_offsets[-1] > 0
        for polls in ("1", None):
            if polls:
                monkeypatch.setenv("GINEX_MOVE_POLLS", polls)
            else:
                monkeypatch.delenv("GINEX_MOVE_POLLS")
            same(want, run())
            same(bare, run(False))
        got, said = found(run, monkeypatch, capfd)
        assert said == [LAUNCHES if cap > most * 2**19 else TOGETHER]
        same(want, got)


def test_most_iterations(ginex, monkeypatch):  # noqa: F811
    rng = np.random.default_rng(0)
    S, n, cap = 2048, 4000, 600
    parts = [rng.permutation(n)[:rng.integers(0, 300)] for _ in range(S)]
    ids = np.concatenate(parts).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
    for policy, ref in (("belady", oracle.changeset), ("lru", oracle.changeset_lru)):
        check_changeset(ginex.changeset(n, dev(ids), off, cap, policy=policy), ref(n, ids, off, cap), (n, ids, off))


# The rows left behind may take the place of those given (final_ids == start_ids), whichever way the lines are found and
# whenever it is given up
@pytest.mark.parametrize("cap,holds_all", [(700, False), (3000, False), (4600, True)])
@pytest.mark.parametrize("planned", ["0", "1", "2"])
@pytest.mark.parametrize("stop", [None, 0, 1, 6, 11])
def test_final_rows_in_the_place_of_the_first(ginex, cap, holds_all, planned, stop, monkeypatch):  # noqa: F811
    from paper_2208_09151_amd import api
    lib, n, S = api._lib.load(), 5000, 12
    rng = np.random.default_rng(cap)
    # (rows of few ids, so that some are accessed again and again)
    parts = [rng.permutation(np.unique((rng.random(900) ** 3 * n).astype(np.int32)))[:600] for _ in range(S)]
    host = np.concatenate(parts).astype(np.int32)
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    start = rng.permutation(n)[:cap].astype(np.int32)
    assert (len(np.unique(host)) <= cap) == holds_all
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
    monkeypatch.setenv("GINEX_PLANNED", planned)
    if stop is not None:
        monkeypatch.setenv("GINEX_MOVE_STOP", str(stop))
    ref = oracle.changeset_resume(n, host, off, cap, start)
    ids, rows, total = dev(host), dev(start), len(host)
    lists = torch.empty(4, total, dtype=torch.int32, device="cuda")
    counts = torch.empty(2 * S + 1, dtype=torch.int64, device="cuda")
    changes = np.zeros(1, dtype=np.int64)
    ws = torch.empty(lib.ginex_changeset_workspace_bytes(n, total, S, cap), dtype=torch.uint8, device="cuda")
    p = api._ptr
    assert lib.ginex_changeset_resume(n, p(ids), api._np_ptr(off), S, cap, p(rows), p(rows), p(lists[0]), p(lists[1]),
                                      p(lists[2]), total, p(counts), p(counts[S + 1:]), p(lists[3]),
                                      api._np_ptr(changes), p(ws), ws.numel(), api._stream()) == 0
    m = int(changes[0])
    assert m > 0
    got = ginex.ChangesetResult(dev(start), lists[0, :m], lists[1, :m], lists[2, :m], counts[:S + 1].cpu().numpy(),
                                counts[S + 1:].cpu().numpy(), np.full(S, cap, dtype=np.int64), rows, lists[3])
    check_resumed(got, ref, (n, host, off))


# Blocks that give up in any iteration leave rows, table and lines as they were, and the call says so
@pytest.mark.parametrize("policy", ["belady", "lru", "resume"])
@pytest.mark.parametrize("cap", [500, 1280, 40_000])          # one block, a few, all
def test_given_up_in_any_iteration(ginex, policy, cap, monkeypatch, capfd):  # noqa: F811
    rng = np.random.default_rng(cap)
    S, n = 10, 3 * cap
    parts = [rng.permutation(n)[:rng.integers(cap // 2, cap + 1)] for _ in range(S)]
    parts[5] = parts[4][::-1].copy()        # every row again in the iteration behind
    ids = np.concatenate(parts).astype(np.int32)
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    start = rng.permutation(n)[:cap].astype(np.int32)
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
    if policy == "resume":
        ref = oracle.changeset_resume(n, ids, off, cap, start)
        run, check = lambda: ginex.changeset_resume(n, dev(ids), off, dev(start)), check_resumed
    else:
        ref = (oracle.changeset if policy == "belady" else oracle.changeset_lru)(n, ids, off, cap)
        run, check = lambda: ginex.changeset(n, dev(ids), off, cap, policy=policy), check_changeset
    for stop, polls, expected in [(None, None, [TOGETHER]), (None, "0", [LAUNCHES])] + \
            [(t, None, [TOGETHER, GIVEN_UP]) for t in (0, 1, S // 2, S - 2, S - 1)] + [(S, None, [TOGETHER])]:
        for name, value in (("GINEX_MOVE_STOP", stop), ("GINEX_MOVE_POLLS", polls)):
            if value is None:
                monkeypatch.delenv(name, raising=False)
            else:
                monkeypatch.setenv(name, str(value))
        got, said = found(run, monkeypatch, capfd)
        assert said == expected, (stop, polls, said)
        check(got, ref, (n, ids, off))


# Calls of several streams at once: one of them has the blocks that wait for each other, the others a launch per iteration
@pytest.mark.parametrize("policy", ["belady", "lru", "resume"])
def test_calls_at_once(ginex, policy, monkeypatch, capfd):  # noqa: F811
    n, S, length, cap, threads = 3_000_000, 60, 60_000, 200_000, 4
    gen = torch.Generator(device="cuda").manual_seed(3)
    work = []
    for _ in range(threads):
        parts = [(torch.rand(length, generator=gen, device="cuda") ** 3 * n).int().clamp(0, n - 1).unique() for _ in range(S)]
        parts = [p[torch.randperm(len(p), generator=gen, device="cuda")] for p in parts]
        work.append((torch.cat(parts), np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)))
    start = torch.randperm(n, generator=gen, device="cuda")[:cap].int()

    def run(k):
        if policy == "resume":
            return ginex.changeset_resume(n, *work[k], start)
        return ginex.changeset(n, *work[k], cap, policy=policy)

    monkeypatch.setenv("GINEX_MOVE_POLLS", "0")
    want = [run(k) for k in range(threads)]
    monkeypatch.setenv("GINEX_MOVE_POLLS", str(1 << 16))      # (no wait ends before the other streams' kernels do)
    torch.cuda.synchronize()

    def one(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(15):
                same(want[k], run(k))
            torch.cuda.current_stream().synchronize()
        return True
    with ThreadPoolExecutor(threads) as pool:
        done, said = found(lambda: list(pool.map(one, range(threads))), monkeypatch, capfd)
    assert all(done) and len(said) == 15 * threads
    assert TOGETHER in said and GIVEN_UP not in said
