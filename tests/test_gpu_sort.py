"""The sort of the accesses around the numbers of words from which its tiles and digits are wider: the lines of a cache
that holds every row, and the rows prefetched by one that holds all but one, against torch (tolerance zero)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import ginex  # noqa: F401

pytestmark = pytest.mark.gpu


# 27 bits in narrow and in wide tiles; 32 bits by 8 and 21 by 7 in wide ones
@pytest.mark.parametrize("total,nodes,validate", [(2**26 - 1, 100_000_000, False), (2**26, 100_000_000, False),
                                                  (2**26 + 16385, 2**25 - 7, False), (2**27 - 1, 2**24, True),
                                                  (2**27 + 3, 2**24, True), (2**27 + 3, 2**21 - 1, False)])
def test_lines_and_first_rows(ginex, total, nodes, validate, monkeypatch):  # noqa: F811
    gen = torch.Generator(device="cuda").manual_seed(total)
    S = max(3, -(-total // (nodes - nodes // 16)))
    off = np.linspace(0, total, S + 1).astype(np.int64)
    rows = torch.randperm(nodes, generator=gen, device="cuda").int()
    longest = int(np.diff(off).max())
    rows = rows[:min(nodes, longest + longest // 20 + 1)].contiguous()
    ids = torch.empty(total, dtype=torch.int32, device="cuda")
    first = torch.full((nodes,), S, dtype=torch.int32, device="cuda")
    for i in range(S):          # a stretch of the rows in another order each time
        n = int(off[i + 1] - off[i])
        at = int(torch.randint(rows.numel(), (1,), generator=gen, device="cuda"))
        step = 2 * (rows.numel() // 3) + 1
        while np.gcd(step, rows.numel()) != 1:
            step += 2
        pick = (torch.arange(n, device="cuda") * step + at) % rows.numel()
        ids[off[i]:off[i + 1]] = rows[pick]
        new = rows[pick].long()
        first[new] = torch.minimum(first[new], torch.tensor(i, dtype=torch.int32, device="cuda"))
    held = torch.nonzero(first < S).flatten()
    order = held[torch.sort(first[held], stable=True)[1]]      # by first access, then id
    line = torch.full((nodes,), -1, dtype=torch.int32, device="cuda")
    line[order] = torch.arange(order.numel(), dtype=torch.int32, device="cuda")
    cap = order.numel()
    if validate:
        monkeypatch.setenv("GINEX_VALIDATE", "1")
    elif 4 * cap >= 3 * total or cap >= nodes - 1:
        cap -= 1                                               # else the rows would not be sorted at all
    cs = ginex.changeset(nodes, ids, off, cap)
    assert torch.equal(cs.init_ids, order[:cap].int())
    if cap == order.numel():
        assert torch.equal(cs.src_line, line[ids.long()])
