"""Evictions of a carried cache that holds the superbatch, all iterations together, against the oracle and the steps on the
bitmap in global memory (tolerance zero): rows that are inserted, die and are evicted again, each wave of them from the lines
of the one before; candidates around the parts a wave takes; more iterations than a wave, or a block, looks at at a time;
evictions around the number that are compared with each other directly; calls that give up on the way."""
import numpy as np
import pytest

import oracle

from test_gpu_parity import check_resumed, dev, ginex  # noqa: F811,F401

pytestmark = pytest.mark.gpu


# new rows of an iteration, iterations, rows held that are never accessed
@pytest.mark.parametrize("new,S,dead", [(1, 3, 1), (1, 63, 1023), (3, 64, 1024), (7, 65, 1025), (256, 9, 2047),
                                        (257, 9, 2049), (1024, 5, 4096), (1025, 6, 5000), (2, 1030, 1500),
                                        (4096, 4, 8200)])
@pytest.mark.parametrize("spread", [False, True])
def test_rows_that_come_and_go(ginex, new, S, dead, spread, monkeypatch):  # noqa: F811
    rng = np.random.default_rng(new * 31 + S)
    n = dead + new * S + 50
    if spread:          # new and old rows anywhere in the order of the ids
        order = rng.permutation(n)
    else:               # the rows of an iteration above all before them: they are evicted as soon as they are dead
        order = np.arange(n)
    start = rng.permutation(order[:dead + 50]).astype(np.int32)
    parts = []
    for t in range(S):
        now = order[dead + 50 + new * t:dead + 50 + new * (t + 1)] if t + 1 < S else order[:0]
        before = parts[-1] if t else order[:0]
        again = before[np.isin(before, order[dead + 50 + new * (t - 1):dead + 50 + new * t])] if t else before
        some = order[dead:dead + 50][rng.random(50) < 0.1]
        parts.append(rng.permutation(np.concatenate([now, again, some])))
    ids = np.concatenate(parts).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
    if len(np.unique(ids)) > len(start):
        more = order[dead + 50:dead + 50 + len(np.unique(ids)) - len(start)]
        start = np.concatenate([start, more]).astype(np.int32)
    ref = oracle.changeset_resume(n, ids, off, len(start), start)
    for way in ("1", "2"):
        monkeypatch.setenv("GINEX_PLANNED", way)
        check_resumed(ginex.changeset_resume(n, dev(ids), off, dev(start)), ref, (n, ids, off))


# The lists' last step gives up in one iteration, while the others' blocks run: the call starts over as any other cache's,
# from the trace or with the loop, and says so
@pytest.mark.parametrize("thresholds", ["0", "1"])
@pytest.mark.parametrize("S", [5, 70])
def test_given_up_in_any_iteration(ginex, S, thresholds, monkeypatch, capfd):  # noqa: F811
    rng = np.random.default_rng(S)
    n, new = 60_000, 300
    order = rng.permutation(n)
    parts = [rng.permutation(order[new * t:new * (t + 2)]) for t in range(S)]       # every row twice, then dead
    ids = np.concatenate(parts).astype(np.int32)
    off = np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)
    start = rng.permutation(order[new * (S + 1) - new // 2:]).astype(np.int32)[:max(new * (S + 1), 8000)]
    ref = oracle.changeset_resume(n, ids, off, len(start), start)
    evicting = np.nonzero(np.diff(ref["cs_offsets"]))[0]
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", thresholds)
    monkeypatch.setenv("GINEX_PLANNED", "1")
    monkeypatch.setenv("GINEX_TRACE", "1")
    for stop in (None, *evicting[[0, 1, len(evicting) // 2, -1]]):
        if stop is not None:
            monkeypatch.setenv("GINEX_PLAN_STOP", str(stop))
        capfd.readouterr()
        check_resumed(ginex.changeset_resume(n, dev(ids), off, dev(start)), ref, (n, ids, off))
        said = capfd.readouterr().err
        assert "planned path\n" in said
        assert ("gave up" in said) == (stop is not None)
        if stop is not None:
            assert f"gave up (reason 3, iteration {stop})" in said
