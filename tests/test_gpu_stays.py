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


# carried caches from 2^22 lines on, of at most as many lines as there are accesses, are dealt by id
# before their rows are marked: both sides of either bound, with (8 M nodes) and without evictions of
# rows that are accessed again, and ids that have to be refused
@pytest.mark.parametrize("cap,total", [(2**22 - 1, 4_800_000), (2**22, 4_800_000), (2**22 + 4097, 2**22 + 4097),
                                       (2**22 + 4097, 2**22 + 4096)])
@pytest.mark.parametrize("n", [8_000_000, 60_000_000])
def test_carried_caches_of_many_lines(ginex, cap, total, n, monkeypatch):  # noqa: F811
    S = 5
    gen = torch.Generator(device="cuda").manual_seed(cap)
    off = np.linspace(0, total, S + 1).astype(np.int64)
    ids = torch.cat([torch.randperm(n, generator=gen, device="cuda")[:k].int() for k in np.diff(off)])
    start = torch.randperm(n, generator=gen, device="cuda")[:cap].int()
    want = None
    for env in ({"GINEX_STATIC_THRESHOLDS": "0", "GINEX_PLANNED": "0"}, {}, {"GINEX_PLANNED": "0"}):
        for name in ("GINEX_STATIC_THRESHOLDS", "GINEX_PLANNED"):
            monkeypatch.setenv(name, env.get(name, "1"))
        got = ginex.changeset_resume(n, ids, off, start)
        want = want or got
        assert np.array_equal(want.miss_count, got.miss_count) and want.miss_count.sum() > 0
        assert np.array_equal(want.cs_offsets, got.cs_offsets)
        for name in ("in_ids", "out_ids", "in_positions", "src_line", "final_ids"):
            assert torch.equal(getattr(want, name), getattr(got, name)), name
        for wrong in (-1, n, int(start[7])):
            bad = start.clone()
            bad[cap // 2] = wrong
            with pytest.raises(ginex.GinexError, match="1 entries of start_ids"):
                ginex.changeset_resume(n, ids, off, bad)
