"""Superbatches whose results go from node order to positions through windows, against the loop over the
cache state (tolerance zero): both sides of the smallest one, a last window of one access and a full one, a last tile
of one access, few and many iterations, room in the workspace that is just enough."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ginex  # noqa: F401

pytestmark = pytest.mark.gpu

LEAST = 2**26


@pytest.mark.parametrize("total,S,n,policy", [
    (LEAST - 1, 9, 20_000_000, "belady"), (LEAST, 9, LEAST // 4, "belady"), (LEAST + 1, 9, LEAST // 4 - 512, "belady"),
    (LEAST + 1, 150, 20_000_000, "belady"), (LEAST + 2**18, 40, 20_000_000, "lru"),
    (LEAST + 2**14 + 1, 700, 60_000_000, "belady"), (5 * 2**25 + 77, 11, 50_000_000, "belady")])
def test_many_accesses(ginex, total, S, n, policy, monkeypatch):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(total % 1009)
    off = np.linspace(0, total, S + 1).astype(np.int64)
    off[2] = off[1]                                     # an empty iteration
    order = torch.randperm(n, generator=gen, device="cuda").int()
    starts = torch.randint(0, n, (S,), generator=gen, device="cuda").tolist()
    pieces = []
    for s, k in zip(starts, np.diff(off)):              # distinct within an iteration
        assert k <= n
        pieces += [order[s:s + k], order[:max(0, s + int(k) - n)]]
    ids = torch.cat(pieces)
    assert ids.numel() == total
    cap = max(int(np.diff(off).max()), n // 8)
    start = torch.randperm(n, generator=gen, device="cuda")[:cap].int()
    runs = [lambda: ginex.changeset(n, ids, off, cap, policy=policy)]
    if policy == "belady":
        runs.append(lambda: ginex.changeset_resume(n, ids, off, start))
    for run in runs:
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "0")
        want = run()
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
        got = run()
        assert np.array_equal(want.miss_count, got.miss_count) and want.miss_count.sum() > 0
        assert np.array_equal(want.cs_offsets, got.cs_offsets) and want.cs_offsets[-1] > 0
        for name in ("in_ids", "out_ids", "in_positions", "src_line"):
            a, b = getattr(want, name), getattr(got, name)
            assert (a is None) == (b is None) and (a is None or torch.equal(a, b)), name
