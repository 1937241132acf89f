"""Belady changesets whose accesses are laid out in more than one window of positions, against the
loop over the cache state (tolerance zero): every list, every line."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ginex  # noqa: F401

pytestmark = pytest.mark.gpu


# 2^25 positions to a window: the last access of the first one, one more, two full ones and a bit
@pytest.mark.parametrize("total", [2**25, 2**25 + 1, 2**26 + 12345])
def test_windows_of_positions(ginex, total, monkeypatch):  # noqa: F811
    n, S = 9_000_000, 9
    gen = torch.Generator(device="cuda").manual_seed(total)
    off = np.linspace(0, total, S + 1).astype(np.int64)
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:k].int() for k in np.diff(off)])
    cap = 8_000_000
    start = torch.randperm(n, generator=gen, device="cuda")[:cap].int()
    for run in (lambda: ginex.changeset(n, ids, off, cap),
                lambda: ginex.changeset_resume(n, ids, off, start)):
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "0")
        want = run()
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
        got = run()
        assert np.array_equal(want.miss_count, got.miss_count) and want.miss_count.sum() > 0
        assert np.array_equal(want.cs_offsets, got.cs_offsets) and want.cs_offsets[-1] > 0
        for name in ("in_ids", "out_ids", "in_positions", "src_line"):
            a, b = getattr(want, name), getattr(got, name)
            assert (a is None) == (b is None) and (a is None or torch.equal(a, b)), name
