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
