"""Results that come to the host through the library's pinned blocks: more calls at once than there are blocks, more
words than one holds, none of them wanted."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest
import torch

import oracle

from test_gpu_parity import check_changeset, dev, ginex  # noqa: F401

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


# Pinned blocks are made where a call needs one and none is free, kept, and not made at all with GINEX_PINNED=0
SCRIPT = """
import os, sys
import numpy as np, torch
import oracle
import paper_2208_09151_amd as g
off = np.arange(9, dtype=np.int64) * 200
ids = np.concatenate([np.random.default_rng(k).permutation(900)[:200] for k in range(8)]).astype(np.int32)
ref = oracle.changeset(900, ids, off, 150)
def call():
    got = g.changeset(900, torch.from_numpy(ids).cuda(), off, 150)
    for name in ("init_ids", "in_ids", "out_ids", "in_positions"):
        assert np.array_equal(getattr(got, name).cpu().numpy(), ref[name]), name
    assert np.array_equal(got.miss_count, ref["miss_count"]) and np.array_equal(got.cs_offsets, ref["cs_offsets"])
    offsets = torch.arange(901, device="cuda", dtype=torch.int64) * 3
    picked = g.sample_superbatch(offsets, torch.arange(2700, device="cuda", dtype=torch.int32) % 900,
                                 torch.arange(40, device="cuda", dtype=torch.int32), np.array([0, 20, 40]), (2, 2))
    assert picked.ids_offsets[-1] > 40
    print("called", file=sys.stderr, flush=True)
os.environ["GINEX_TRACE"] = "2"
os.environ["GINEX_PINNED"] = "0"
call()
assert not hasattr(g.api._staging, "buffer")
del os.environ["GINEX_PINNED"]
call()
assert hasattr(g.api._staging, "buffer")
call()
"""


def test_pinned_memory(ginex):  # noqa: F811
    run = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr
    without, made, kept = run.stderr.split("called")[:3]
    assert "pinned" not in without and "pinned" not in kept
    assert made.count("[ginex] pinned block 1 of at most 16") == made.count("pinned block") == 1


# The thread's buffer is made by its first call, in whatever mode that one runs, and serves all of them
@pytest.mark.parametrize("first,then", [(True, False), (False, True)])
def test_modes_of_the_first_call(ginex, first, then):  # noqa: F811
    ids, off = trace(5, 8, 900, 200)
    ref = oracle.changeset(900, ids, off, 150)

    def calls():
        for special in (first, then, first):
            with torch.inference_mode(special), torch.device("cuda" if special else "cpu"):
                got = ginex.changeset(900, dev(ids), off, 150)
            check_changeset(got, ref, (900, ids, off))
        return True
    with ThreadPoolExecutor(1) as pool:
        assert pool.submit(calls).result()
