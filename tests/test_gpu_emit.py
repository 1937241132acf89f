"""Where the sampler's bucket hops put their results: numbers of batches and tiles around the limits at which
the sums in front of a batch or tile come from a launch of their own, seeds and their offsets around what fits
LDS and a launch's arguments, one hop only, hops through the tables in between.  Everything is compared with
the oracle element by element (tolerance zero)."""
import numpy as np
import pytest

import oracle

from test_gpu_buckets import both
from test_gpu_parity import dev, ginex, small_graph  # noqa: F401

pytestmark = pytest.mark.gpu


def distinct(n, sizes, seed=0):
    rng = np.random.default_rng(seed)
    return [rng.choice(n, size=m, replace=False) for m in sizes]


@pytest.mark.parametrize("fanout", [(3,), (2, 3), (2, 2, 2)])
@pytest.mark.parametrize("S", [1, 2, 255, 256, 257, 1024, 1025])
def test_numbers_of_batches(ginex, S, fanout):  # noqa: F811
    off, ind = small_graph(n=900, e=6000)
    sizes = np.random.default_rng(S).integers(0, 9, S)
    both(ginex, off.numpy(), ind.numpy(), distinct(900, sizes), fanout)


# 1 024 seeds and their picks beside them, more picks, 12 288 seeds in LDS, one more; repeated seeds
@pytest.mark.parametrize("seeds,k", [(1024, 11), (1024, 12), (1025, 2), (12288, 2), (12289, 2)])
def test_seeds_around_what_fits_lds(ginex, seeds, k):  # noqa: F811
    off, ind = small_graph(n=20_000, e=100_000)
    batches = distinct(20_000, (seeds, 0, 5)) + [np.random.default_rng(1).integers(0, 700, seeds)]
    both(ginex, off.numpy(), ind.numpy(), batches, (k, 2))


@pytest.mark.parametrize("nodes", [262_144, 262_145, 300_000])
def test_tiles_around_what_a_block_adds_up(ginex, nodes):  # noqa: F811
    """The list of the second hop holds every node of the graph: 1 024 tiles, or more."""
    off = np.arange(nodes + 1, dtype=np.int64) * 32
    ind = np.concatenate([np.arange(i, i + nodes * 32, 32) % nodes for i in range(32)]).reshape(32, nodes).T.copy()
    ind = ((ind + np.arange(32) * 9973 + np.arange(nodes)[:, None] * 31) % nodes).astype(np.int32).ravel()
    both(ginex, off, ind, distinct(nodes, (12_000, 7)), (32, 32, 2))


@pytest.mark.parametrize("fanout", [(3, 33, 2), (33, 3, 2), (3, 2, 33), (3, 33)])
def test_hops_through_the_tables_in_between(ginex, fanout):  # noqa: F811
    off, ind = small_graph(n=5000, e=200_000)
    both(ginex, off.numpy(), ind.numpy(), distinct(5000, (40, 0, 300, 1)), fanout)


@pytest.mark.parametrize("fanout", [(4,), (4, 3), (20, 3)])
def test_ids_without_adjacency(ginex, fanout):  # noqa: F811
    off, ind = small_graph(n=5000, e=60_000)
    batches = distinct(5000, (700, 0, 1000, 3))
    seeds = np.concatenate(batches).astype(np.int32)
    so = np.cumsum([0] + [len(b) for b in batches])
    ref = oracle.sample_superbatch(off.numpy(), ind.numpy(), seeds, so, fanout, rng_seed=5, first_batch_index=2)
    res = ginex.sample_superbatch(off.cuda(), ind.cuda(), dev(seeds), so, fanout, rng_seed=5, first_batch_index=2,
                                  with_adj=False)
    assert np.array_equal(res.ids.cpu().numpy(), ref["ids"])
    assert np.array_equal(res.ids_offsets, ref["ids_offsets"])
    assert np.array_equal(res.hop_sizes.ravel(), np.asarray(ref["hop_sizes"]).ravel())
