"""A cache that holds every row with wide tiles (16 384 accesses, from 512 of them and 1 024 buckets on) and with narrow ones:
full tiles, one more or less, empty iterations, few and many buckets, ids in order, a share longer than a wave takes at
once; against the sorted accesses (tolerance zero)."""
import numpy as np
import pytest
import torch

from test_gpu_fits import same, trace
from test_gpu_parity import ginex  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [(16384,) * 512, (16384,) * 511, (16383, 16385) * 128, (0, 32769, 1, 0) * 64,
                                     (49_153,) * 128])
@pytest.mark.parametrize("n", [2_097_153, 2_095_104, 30_000_001])
def test_lengths_around_wide_tiles(ginex, n, lengths, monkeypatch):  # noqa: F811
    ids, off = trace(n, lengths, n)
    same(ginex, n, ids, off, n, monkeypatch)


@pytest.mark.parametrize("order", ["mixed", "sorted"])
def test_long_shares_of_wide_tiles(ginex, order, monkeypatch):  # noqa: F811
    n, S = 1 << 26, 520
    gen = torch.Generator(device="cuda").manual_seed(3)
    parts = []
    for i in range(S):
        near = torch.randperm(1 << 15, generator=gen, device="cuda")[:(0, 200, 16_000 if i < 40 else 17, 1)[i % 4]]
        far = (1 << 15) + (torch.arange(300, device="cuda") * 200_003 + i * 7919) % (n - (1 << 15))
        ids = torch.cat([near, far]).int()
        parts.append(ids.sort()[0] if order == "sorted" else ids[torch.randperm(len(ids), generator=gen, device="cuda")])
    off = np.concatenate([[0], np.cumsum([len(x) for x in parts])]).astype(np.int64)
    same(ginex, n, torch.cat(parts), off, int(off[-1]), monkeypatch)
