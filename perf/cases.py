"""The cases by which the speed of the library is measured: the calls a training pipeline makes
for a superbatch, through the Python entry points, from the smallest workload to the largest.

Graphs and traces follow the R-MAT marginals of the workloads in ``workload/`` (every bit of a
node's label is set with probability ``skew``, ids relabelled by an affine bijection), drawn
directly on the GPU so that inputs of any seed are ready in well under a second or two.
Everything the library returns is whole numbers or copied bytes: the tolerance is exact.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2208_09151_amd as ginex

TABLE_BITS = 20         # uniform bits that pick one block of label bits


def listed():
    return [
        # Superbatch sampling.  The smallest workload: launches and host round trips count.
        dict(name="sample-16k", kind="sample", nodes=16384, edges=262144, skew=0.24, batch=256,
             batches=8, last=102, fanout="10,10,10", wide=False),
        # an ordinary graph with int32 offsets, 3 hops
        dict(name="sample-1M", kind="sample", nodes=1 << 20, edges=16 << 20, skew=0.24, batch=1000,
             batches=20, last=1000, fanout="10,10,10", wide=False),
        # two wide hops, an odd number of nodes and seeds, a short last batch, int64 offsets
        dict(name="sample-3M-two-hops", kind="sample", nodes=3_000_017, edges=60_000_011, skew=0.30,
             batch=777, batches=33, last=301, fanout="25,10", wide=True),
        # the large power-law graph: 200 batches of 1000 seeds at once
        dict(name="sample-111M", kind="sample", nodes=111_000_000, edges=1_600_000_000, skew=0.24,
             batch=1000, batches=200, last=1000, fanout="10,10,10", wide=True),
        # Changeset precomputation.  The smallest workload, a cache smaller than one iteration.
        dict(name="changeset-16k", kind="changeset", nodes=16384, batches=8, length=3500, skew=0.24,
             cap=2048, policy="belady"),
        # the policy Belady's is compared with, on an ordinary trace and a cache of 10 % of the rows
        dict(name="changeset-1M-lru", kind="changeset", nodes=1 << 20, batches=20, length=76_000,
             skew=0.24, cap=104_857, policy="lru"),
        # the large graph with a cache that holds every row of the superbatch ...
        dict(name="changeset-111M-fits", kind="changeset", nodes=111_000_000, batches=200,
             length=177_000, skew=0.24, cap=27_750_000, policy="belady"),
        # ... and with one that holds a sixteenth of them, so that every iteration evicts
        dict(name="changeset-111M-pressure", kind="changeset", nodes=111_000_000, batches=200,
             length=177_000, skew=0.24, cap=573_000, policy="belady"),
        # the social-graph shape: long iterations, a cache of 20 % of the rows that is too small
        dict(name="changeset-65M-long", kind="changeset", nodes=65_600_000, batches=200,
             length=820_000, skew=0.33, cap=13_120_000, policy="belady"),
        # a cache carried over from the superbatch before: changesets from its state
        dict(name="resume-111M", kind="resume", nodes=111_000_000, batches=200, length=177_000,
             skew=0.24, cap=27_750_000),
        # The main loop on resident rows of 512 bytes, lines resolved by the changeset stage.
        dict(name="gather-resident", kind="gather", nodes=4_000_000, dim=128, batches=20,
             length=177_000, skew=0.24, cap=4_000_000, start=False),
        # One whole superbatch of the ordinary workload: sampling, changesets, cache
        # initialization and the main loop with misses and updates (features in pinned memory).
        dict(name="superbatch-1M", kind="superbatch", nodes=1 << 20, edges=16 << 20, skew=0.24,
             batch=1000, batches=20, last=1000, fanout="10,10,10", wide=False, dim=128,
             cap=104_857),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sample", "sample", "changeset", "changeset", "resume", "gather",
                       "superbatch"])
    skew = round(rng.uniform(0.22, 0.36), 3)
    if kind in ("sample", "superbatch"):
        nodes = _log(rng, 10_000, 30_000_000 if kind == "sample" else 2_000_000)
        batch = _log(rng, 50, 1000)
        case = dict(kind=kind, nodes=nodes, edges=int(nodes * rng.uniform(6, 32)), skew=skew,
                    batch=batch, batches=_log(rng, 1, 100 if kind == "sample" else 20),
                    last=rng.randint(1, batch),
                    fanout=rng.choice(["10,10,10", "10,10,10", "25,10", "15,10,5", "10,10", "5,5,5"]),
                    wide=rng.random() < 0.5)
        if kind == "superbatch":
            case["dim"] = 4 * rng.randint(8, 48)
            case["cap"] = max(1, int(nodes * rng.uniform(0.02, 0.5)))
        return case
    if kind == "gather":
        nodes = _log(rng, 10_000, 2_000_000)
        batches = _log(rng, 2, 20)
        length = _log(rng, 300, min(170_000, nodes // 8))
        start = rng.random() < 0.5
        cap = max(1, int(nodes * rng.uniform(0.02, 0.5))) if start else nodes
        return dict(kind=kind, nodes=nodes, dim=4 * rng.randint(4, 64), batches=batches,
                    length=length, skew=skew, cap=cap, start=start)
    nodes = _log(rng, 10_000, 60_000_000)
    batches = _log(rng, 2, 256)
    length = _log(rng, 300, min(400_000, nodes // 8, 40_000_000 // batches))
    rows = _distinct(nodes, skew, _draws(nodes, skew, length) * batches)
    if kind == "changeset":
        share = math.exp(rng.uniform(math.log(0.01), math.log(1.3)))
        return dict(kind=kind, nodes=nodes, batches=batches, length=length, skew=skew,
                    cap=max(1, int(rows * share)),
                    policy="lru" if rng.random() < 0.25 else "belady")
    share = math.exp(rng.uniform(math.log(0.03), math.log(3)))
    return dict(kind=kind, nodes=nodes, batches=batches, length=length, skew=skew,
                cap=max(1, min(nodes, int(rows * share))))


# ---- expected sizes (for work() and for the caches of drawn cases) ---------------------------

def _levels(nodes, skew):
    """(number of labels, probability of one) per count of set bits."""
    bits = max(1, (nodes - 1).bit_length())
    shrink = nodes / 2 ** bits      # labels beyond the last node are folded back
    return [(math.comb(bits, k) * shrink, (1 - skew) ** (bits - k) * skew ** k / shrink)
            for k in range(bits + 1)]


def _distinct(nodes, skew, draws):
    return sum(c * -math.expm1(-draws * p) for c, p in _levels(nodes, skew))


def _draws(nodes, skew, length):
    """How many draws give `length` distinct ids (and a margin, the surplus is left out)."""
    want = length + 4 * math.sqrt(length) + 8
    lo, hi = length, 2 * length
    while _distinct(nodes, skew, hi) < want:
        hi *= 2
    while hi - lo > 1 + lo // 1000:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if _distinct(nodes, skew, mid) >= want else (mid, hi)
    return hi


def _lengths(case):
    """Accesses per iteration: ragged, up to an eighth below `length`."""
    n = case["length"]
    return [n - i * 7919 % (n // 8 + 1) for i in range(case["batches"])]


def _mean_picks(case, k, weighted):
    """Mean of min(degree, k) over the nodes, or over the ends of edges."""
    total = 0.0
    for c, p in _levels(case["nodes"], case["skew"]):
        lam = case["edges"] * p
        below = 0.0
        if lam < 60 + 2 * k:
            q = math.exp(-lam)
            for d in range(k):
                below += q * (k - d)
                q *= lam / (d + 1)
        total += (c * p if weighted else c / case["nodes"]) * (k - below)
    return total


def _rows(case):
    """Expected distinct rows of the superbatch's accesses."""
    if "fanout" in case:
        draws = _sample_sizes(case)[2]
    else:
        draws = case["batches"] * _draws(case["nodes"], case["skew"], case["length"])
    return _distinct(case["nodes"], case["skew"], draws)


def _sample_sizes(case):
    """Expected ids, frontier rows and edges of a superbatch."""
    seeds = (case["batches"] - 1) * case["batch"] + case["last"]
    per = seeds / case["batches"]
    drawn, rows, edges = 0.0, 0.0, 0.0
    for k in _fanout(case):
        found = _distinct(case["nodes"], case["skew"], drawn) if drawn else 0.0
        picks = per * _mean_picks(case, k, False) + found * _mean_picks(case, k, True)
        rows += per + found + 1
        edges += picks
        drawn += picks
    ids = min(per + _distinct(case["nodes"], case["skew"], drawn), case["nodes"])
    return ids * case["batches"], rows * case["batches"], edges * case["batches"]


def work(case):
    kind = case["kind"]
    total = 0.0
    if kind in ("sample", "superbatch"):
        ids, rows, edges = _sample_sizes(case)
        # the rows' offsets and the picked neighbours are read, ids, row pointers and columns written
        total += rows * ((16 if case["wide"] else 8) + 8) + edges * (4 + 4) + ids * 4
        accesses = ids
    else:
        accesses = sum(_lengths(case))
    if kind in ("changeset", "resume", "superbatch"):
        total += accesses * (4 + 4)                 # ids in, lines out
        rows = _rows(case)
        if kind == "resume":
            total += 2 * 4 * case["cap"]            # start and final state
        else:
            total += 4 * min(case["cap"], rows)     # C_0
        if case["cap"] < rows:
            total += 12 * 0.1 * accesses            # about one access in ten changes the cache
    if kind in ("gather", "superbatch"):
        total += accesses * (8 + 2 * 4 * case["dim"])
        if case.get("start", kind == "superbatch"):
            total += case["cap"] * (8 + 2 * 4 * case["dim"])
    return {"bytes": int(total), "flops": 0}


def tolerance(case):
    return "exact"


# ---- inputs ------------------------------------------------------------------------------------

def _fanout(case):
    return [int(k) for k in case["fanout"].split(",")]


class _Labels:
    """Draws node ids with the R-MAT marginal: label bits set with probability ``skew``, three
    blocks of bits looked up per random word, labels scattered by an affine bijection."""

    def __init__(self, nodes, skew, seed):
        self.nodes = nodes
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)
        bits = max(1, (nodes - 1).bit_length())
        widths = [bits // 3 + (i < bits % 3) for i in range(3)]
        self.tables, self.shifts = [], []
        at = 0
        for w in widths:
            value = torch.arange(1 << w, dtype=torch.int64)
            ones = torch.zeros(1 << w, dtype=torch.float64)
            for b in range(w):
                ones += (value >> b) & 1
            p = (1 - skew) ** (w - ones) * skew ** ones
            edge = torch.cumsum(p, 0)
            u = (torch.arange(1 << TABLE_BITS, dtype=torch.float64) + 0.5) / (1 << TABLE_BITS)
            pick = torch.searchsorted(edge, u).clamp_(max=(1 << w) - 1)
            self.tables.append((pick << at).cuda())
            at += w
        mul = (0x9E3779B97F4A7C15 ^ (seed * 0xD1B54A32D192ED03)) % nodes | 1
        while math.gcd(mul, nodes) != 1:
            mul += 2
        self.mul = mul % nodes if nodes > 1 else 0
        self.add = (seed * 0xBF58476D1CE4E5B9 + 12345) % nodes

    def words(self, n):
        return torch.empty(n, dtype=torch.int64, device="cuda").random_(generator=self.gen)

    def ids(self, n):
        w = self.words(n)
        mask = (1 << TABLE_BITS) - 1
        label = self.tables[0][w & mask]
        label |= self.tables[1][(w >> TABLE_BITS) & mask]
        label |= self.tables[2][(w >> 2 * TABLE_BITS) & mask]
        return (label % self.nodes * self.mul + self.add) % self.nodes


def _graph(case, labels):
    """CSR: a row's length and the entries of the rows follow the same marginal."""
    nodes, edges = case["nodes"], case["edges"]
    degree = torch.zeros(nodes, dtype=torch.int64, device="cuda")
    indices = torch.empty(edges, dtype=torch.int32, device="cuda")
    chunk = 1 << 26
    for lo in range(0, edges, chunk):
        n = min(chunk, edges - lo)
        degree += torch.bincount(labels.ids(n), minlength=nodes)
        indices[lo:lo + n] = labels.ids(n)
    offsets = torch.zeros(nodes + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(degree, 0, out=offsets[1:])
    return (offsets if case["wide"] else offsets.to(torch.int32)), indices


def _seeds(case, labels):
    """Distinct training nodes, `batch` to a batch, the last batch short."""
    sizes = [case["batch"]] * (case["batches"] - 1) + [case["last"]]
    offsets = np.zeros(len(sizes) + 1, dtype=np.int64)
    np.cumsum(sizes, out=offsets[1:])
    step = 2 * (labels.nodes // 3) + 1
    while math.gcd(step, labels.nodes) != 1:
        step += 2
    at = torch.arange(int(offsets[-1]), dtype=torch.int64, device="cuda")
    first = int(labels.words(1)[0]) % labels.nodes
    return ((at * step + first) % labels.nodes).to(torch.int32), offsets


def _trace(case, labels):
    """Access trace: per iteration a fixed number of distinct ids in random order."""
    S, draws = case["batches"], _draws(case["nodes"], case["skew"], case["length"])
    lengths = torch.tensor(_lengths(case), device="cuda")
    step = max(1, (1 << 26) // draws)
    parts = []
    for lo in range(0, S, step):
        n = min(step, S - lo)
        which = torch.arange(n, device="cuda").repeat_interleave(draws)
        key = torch.sort(which << 32 | labels.ids(n * draws))[0]
        key = torch.unique_consecutive(key)
        which = key >> 32
        order = torch.sort(which << 40 | labels.words(key.numel()) & ((1 << 40) - 1))[1]
        found = torch.bincount(which, minlength=n)
        if not bool((found >= lengths[lo:lo + n]).all()):
            raise RuntimeError("too few distinct ids were drawn")
        at = torch.arange(key.numel(), device="cuda") - (torch.cumsum(found, 0) - found)[which]
        kept = order[at < lengths[lo + which]]
        parts.append((key & 0xFFFFFFFF).to(torch.int32)[kept])
    offsets = np.zeros(S + 1, dtype=np.int64)
    np.cumsum(_lengths(case), out=offsets[1:])
    return torch.cat(parts), offsets


def _carried(case, labels):
    """The state earlier superbatches left: the rows they accessed, filled up from the lower end
    of the ids (the largest dead ids leave first), in no particular line order."""
    nodes, cap = labels.nodes, case["cap"]
    held = torch.zeros(nodes, dtype=torch.bool, device="cuda")
    for _ in range(6):
        left = case["batches"] * _draws(case["nodes"], case["skew"], case["length"])
        while left > 0:
            n = min(left, 1 << 26)
            held[labels.ids(n)] = True
            left -= n
    rows = torch.nonzero(held).flatten()
    if rows.numel() < cap:
        rest = torch.nonzero(~held).flatten()[:cap - rows.numel()]
        rows = torch.cat([rows, rest])
    order = torch.sort(labels.words(rows.numel()))[1][:cap]
    return rows[order].to(torch.int32)


def _features(nodes, dim, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1)
    out = torch.empty((nodes, dim), dtype=torch.float32, pin_memory=True)
    chunk = max(1, (1 << 28) // dim)
    for lo in range(0, nodes, chunk):
        n = min(chunk, nodes - lo)
        out[lo:lo + n].copy_(torch.randn((n, dim), generator=gen, device="cuda"))
    return out


def _zeros(n, dtype=torch.int32):
    return torch.zeros(n, dtype=dtype, device="cuda")


def prepare(case, seed):
    labels = _Labels(case["nodes"], case["skew"], seed)
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind in ("sample", "superbatch"):
        s["offsets"], s["indices"] = _graph(case, labels)
        s["seeds"], s["seed_offsets"] = _seeds(case, labels)
        s["fanout"] = _fanout(case)
        s["rng_seed"] = seed & 0xFFFF
    else:
        s["ids"], s["ids_offsets"] = _trace(case, labels)
    if kind == "resume":
        s["start_ids"] = _carried(case, labels)
    # The program's own buffers, used superbatch after superbatch: what the sampler writes and
    # the lists that wait for the executor.
    if kind in ("sample", "superbatch"):
        ids, rows, edges = (int(1.5 * n) + 10_000 for n in _sample_sizes(case))
        s["buffers"] = _zeros(ids), _zeros(rows, torch.int64), _zeros(edges)
    else:
        ids = s["ids"].numel()
    if kind in ("changeset", "resume", "superbatch"):
        s["lists"] = {"init_ids": _zeros(case["cap"]), "in_ids": _zeros(ids),
                      "out_ids": _zeros(ids), "in_positions": _zeros(ids)}
    if kind == "superbatch":
        s["lists"]["src_line"] = _zeros(ids)
    if kind in ("gather", "superbatch"):
        s["slow"] = _features(case["nodes"], case["dim"], seed)
        s["cache"] = ginex.FeatureCache(s["slow"], case["cap"])
        s["inputs"] = torch.zeros((ids, case["dim"]), dtype=torch.float32, device="cuda")
    if kind == "gather":
        s["cs"] = ginex.changeset(case["nodes"], s["ids"], s["ids_offsets"], case["cap"])
        if not case["start"]:
            s["cache"].init(s["cs"].init_ids)
    return s


def _sample(s):
    return ginex.sample_superbatch(s["offsets"], s["indices"], s["seeds"], s["seed_offsets"],
                                   s["fanout"], rng_seed=s["rng_seed"], first_batch_index=3,
                                   out=s["buffers"])


def _main_loop(cache, ids, ids_offsets, cs, inputs):
    """Every iteration's batch input: gather, then the cache update of the iteration."""
    io, co, slow = ids_offsets.tolist(), cs.cs_offsets.tolist(), cs.miss_count.tolist()
    for i in range(len(io) - 1):
        at, ch = slice(io[i], io[i + 1]), slice(co[i], co[i + 1])
        cache.gather(ids[at], inputs[at], cs.in_ids[ch], cs.out_ids[ch], cs.in_positions[ch],
                     src_line=cs.src_line[at], n_slow=slow[i])


def _keep(s, cs):
    """The lists of a superbatch put where its executor will read them."""
    out = {"cs_offsets": cs.cs_offsets, "miss_count": cs.miss_count, "init_ready": cs.init_ready,
           "src_line": cs.src_line}
    for name, buffer in s["lists"].items():
        made = getattr(cs, name)
        buffer[:made.numel()].copy_(made)
        out[name] = buffer
    return out


def _sampled(s, r):
    ids, rowptr, col = s["buffers"]
    return {"ids": ids, "adj_rowptr": rowptr, "adj_col": col, "ids_offsets": r.ids_offsets,
            "hop_sizes": r.hop_sizes, "adj_row_offsets": r.adj_row_offsets,
            "adj_col_offsets": r.adj_col_offsets}


def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "sample":
        return _sampled(s, _sample(s))
    if kind == "changeset":
        return _keep(s, ginex.changeset(c["nodes"], s["ids"], s["ids_offsets"], c["cap"],
                                        policy=c["policy"]))
    if kind == "resume":
        cs = ginex.changeset_resume(c["nodes"], s["ids"], s["ids_offsets"], s["start_ids"])
        return dict(_keep(s, cs), final_ids=cs.final_ids)
    if kind == "gather":
        if c["start"]:
            s["cache"].init(s["cs"].init_ids)
        _main_loop(s["cache"], s["ids"], s["ids_offsets"], s["cs"], s["inputs"])
        return s["inputs"]
    r = _sample(s)
    cs = ginex.changeset(c["nodes"], r.ids, r.ids_offsets, c["cap"])
    s["cache"].init(cs.init_ids)
    _main_loop(s["cache"], r.ids, r.ids_offsets, cs, s["inputs"])
    return {"sample": _sampled(s, r), "changesets": _keep(s, cs), "inputs": s["inputs"],
            "addr": s["cache"].addr}


def exact(case, seed):
    """A gathered row is the row of the feature table; the other outputs are whole numbers."""
    if case["kind"] != "gather":
        return None
    labels = _Labels(case["nodes"], case["skew"], seed)
    ids, _ = _trace(case, labels)
    table = _features(case["nodes"], case["dim"], seed)
    return table[ids.cpu().long()]
