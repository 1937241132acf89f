"""Results that come to the host through the library's pinned blocks: more calls at once than there are blocks, more
words than one holds."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu


def trace(seed, S, n, most):
    rng = np.random.default_rng(seed)
    parts = [rng.permutation(n)[:rng.integers(0, most + 1)] for _ in range(S)]
    return np.concatenate(parts).astype(np.int32), np.cumsum([0] + [len(p) for p in parts]).astype(np.int64)


def test_more_calls_at_once_than_blocks(ginex):  # noqa: F811
    def one(k):
        ids, off = trace(k, 30, 500, 40)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got = ginex.changeset(500, dev(ids), off, 60 + k)
                check_changeset(got, oracle.changeset(500, ids, off, 60 + k), (500, ids, off))
        return True
    with ThreadPoolExecutor(24) as pool:
        assert all(pool.map(one, range(24)))


# the offsets of 8 191 iterations are 64 KB, together with their rows of C_0 more than a block holds
@pytest.mark.parametrize("S", [4090, 8191])
def test_more_words_than_a_block(ginex, S):  # noqa: F811
    ids, off = trace(S, S, 300, 5)
    got = ginex.changeset(300, dev(ids), off, 40)
    check_changeset(got, oracle.changeset(300, ids, off, 40), (300, ids, off))
