"""The smallest Belady calls in one workgroup, against the oracle (tolerance zero): numbers of rows and iterations
around what it takes, iterations around its threads, caches of one line to all rows but one, too little room."""
import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu


def trace(rng, rows, n, lengths):
    """Every one of `rows` ids of n is accessed if the iterations have room for them."""
    ids = np.sort(rng.choice(n, size=rows, replace=False))
    left, parts = list(rng.permutation(rows)), []
    for k in lengths:
        new, left = left[:k // 2], left[k // 2:]
        rest = np.setdiff1d(np.arange(rows), new)
        parts.append(rng.permutation(np.concatenate([new, rng.choice(rest, size=k - len(new), replace=False)])))
    return ids[np.concatenate(parts).astype(int)].astype(np.int32), np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


@pytest.mark.parametrize("rows,n,lengths", [
    (1, 1, (1, 1, 1)), (2, 9, (1, 2, 0, 1)), (63, 70, (40,) * 5), (64, 64, (64, 0, 64, 1)), (65, 1000, (33,) * 9),
    (1023, 2000, (1000, 1023, 5, 700)), (1024, 1024, (1024,) * 3), (1025, 1 << 20, (1025, 1024, 1023) * 2),
    (2000, 2000, (90,) * 255), (2000, 2000, (90,) * 256), (2000, 2000, (90,) * 257),
    (12287, 16384, (5000,) * 6), (12288, 16384, (5000,) * 6), (12289, 16384, (5000,) * 6),
    (12288, 12288, (12288,) * 3), (9000, 1 << 26, (2048, 2049, 1) * 9)])
def test_around_the_limits(ginex, rows, n, lengths):  # noqa: F811
    rng = np.random.default_rng(rows + len(lengths))
    ids, off = trace(rng, rows, n, lengths)
    distinct = len(np.unique(ids))
    for cap in sorted({1, 2, max(1, distinct // 9), max(1, distinct // 2), distinct - 1, distinct}):
        if cap < 1:
            continue
        ref = oracle.changeset(n, ids, off, cap)
        check_changeset(ginex.changeset(n, dev(ids), off, cap), ref, (n, ids, off))


@pytest.mark.parametrize("seed", range(6))
def test_random_traces(ginex, seed):  # noqa: F811
    rng = np.random.default_rng(seed)
    for _ in range(12):
        n = int(rng.integers(2, 9000))
        S = int(rng.integers(1, 40))
        most = int(rng.integers(1, min(n, 3000) + 1))
        weights = rng.random(n) ** int(rng.integers(1, 9)) + 1e-9
        parts = [rng.choice(n, size=int(rng.integers(0, most + 1)), replace=False, p=weights / weights.sum())
                 for _ in range(S)]
        ids = np.concatenate(parts).astype(np.int32)
        off = np.concatenate([[0], np.cumsum([len(p) for p in parts])]).astype(np.int64)
        if len(ids) == 0:
            continue
        cap = int(rng.integers(1, len(np.unique(ids)) + 1))
        check_changeset(ginex.changeset(n, dev(ids), off, cap), oracle.changeset(n, ids, off, cap), (n, ids, off))
        got = ginex.changeset(n, dev(ids), off, cap, with_lines=False)
        assert got.src_line is None
