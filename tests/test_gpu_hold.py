"""The rows of a large carried cache, put together a stretch of ids at a time in LDS (from 2^22 lines on, up to 2^27 nodes) or
as bytes (beyond), against the loop over the state, which does neither (tolerance zero), and rows that are refused, more
lines than nodes among them."""
import numpy as np
import pytest
import torch

import paper_2208_09151_amd
from test_gpu_parity import ginex  # noqa: F401

pytestmark = pytest.mark.gpu

NAMES = ("in_ids", "out_ids", "in_positions", "src_line", "final_ids")


# every row held, stretches of 2^16 ids; a last stretch of three ids; 2^19; beyond; fewer lines than are dealt
@pytest.mark.parametrize("nodes,cap", [(2**22, 2**22), (2**23 + 3, 2**22 + 5), (2**24 + 65537, 2**22),
                                       (2**27, 2**23 - 1), (2**27 + 1, 2**22), (2**23, 2**22 - 1)])
@pytest.mark.parametrize("low", [False, True])
def test_carried_rows(ginex, nodes, cap, low, monkeypatch):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(nodes + low)
    S, length = 3, 1_500_000

    def some(n, most=nodes):
        step = 2 * (most // 3) + 1
        while np.gcd(step, most) != 1:
            step += 2
        at = int(torch.randint(most, (1,), generator=gen, device="cuda"))
        return ((torch.arange(n, device="cuda") * step + at) % most).int()

    parts = [some(length), some(length)]
    again = parts[0][:length // 2]                    # the third: half of the first, and rows that are not among them
    other = some(min(nodes, 2 * length))
    parts.append(torch.cat([again, other[~torch.isin(other, again)][:length - length // 2]]))
    ids = torch.cat(parts)
    off = np.arange(S + 1, dtype=np.int64) * length
    rows = torch.arange(cap, device="cuda", dtype=torch.int32) if low else some(cap)
    start = rows[torch.randperm(cap, generator=gen, device="cuda")]
    monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "0")
    monkeypatch.setenv("GINEX_PLANNED", "0")
    ref = ginex.changeset_resume(nodes, ids, off, start)
    for planned in ("1", "0"):
        monkeypatch.setenv("GINEX_STATIC_THRESHOLDS", "1")
        monkeypatch.setenv("GINEX_PLANNED", planned)
        got = ginex.changeset_resume(nodes, ids, off, start)
        assert np.array_equal(got.miss_count, ref.miss_count) and np.array_equal(got.cs_offsets, ref.cs_offsets)
        for name in NAMES:
            assert torch.equal(getattr(got, name), getattr(ref, name)), name
    for bad in (nodes, -1, int(start[1])):
        broken = start.clone()
        broken[0] = bad
        with pytest.raises(paper_2208_09151_amd.GinexError):
            ginex.changeset_resume(nodes, ids, off, broken)


# more lines than there are nodes: some row is there twice, whatever the rows are, and the call says so
@pytest.mark.parametrize("nodes", [3000, 40_000, 65_536, 65_537])
def test_more_lines_than_nodes(ginex, nodes):  # noqa: F811
    cap = 2**22
    length = nodes - 1
    S = -(-cap // length)
    gen = torch.Generator(device="cuda").manual_seed(nodes)
    ids = torch.cat([torch.randperm(nodes, generator=gen, device="cuda")[:length].int() for _ in range(S)])
    start = torch.randint(nodes, (cap,), generator=gen, device="cuda").int()
    with pytest.raises(paper_2208_09151_amd.GinexError, match="out of range or repeated"):
        ginex.changeset_resume(nodes, ids, np.arange(S + 1, dtype=np.int64) * length, start)
    # (and the next call finds nothing of it)
    off = np.arange(3, dtype=np.int64) * length
    got = ginex.changeset_resume(nodes, ids[:2 * length], off, torch.arange(nodes, device="cuda").int())
    assert got.miss_count.sum() == 0
