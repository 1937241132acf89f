"""The rule by which the GPU path lays out every Belady changeset before it assigns a single
cache line (Section 3.4's recurrence): with the threshold bucket j*_t and the number of rows to
drop from it known for every iteration t, the stay of a row between two accesses i and j ends
at the first t in [i, j) with j*_t < j; where j*_t = j the row is in the bucket that is cut, and
only there the class (incoming rows first) and the id decide.  Cuts of different iterations
depend on each other only through the accesses of the iteration (bucket t) and earlier cuts of
the same bucket.  Written out here in numpy, sharing no code with the kernels, and compared with
the oracle: misses, insertions, evictions, cache lines."""
import numpy as np
import pytest

import oracle


def thresholds(off, nxt, S, start_keys):
    R = np.bincount(start_keys, minlength=S + 1)
    out = []
    for t in range(S):
        C = R.copy()
        drop = int(off[t + 1] - off[t] - C[t])
        C[:t + 1] = 0
        C += np.bincount(nxt[off[t]:off[t + 1]], minlength=S + 1)
        jstar, rem, cum = S + 1, 0, 0
        if drop > 0:
            for j in range(S, t, -1):
                if cum <= drop < cum + C[j]:
                    jstar, rem = j, drop - cum
                    break
                cum += C[j]
        R = np.where(np.arange(S + 1) < jstar, C, 0)
        if jstar <= S:
            R[jstar] = C[jstar] - rem
        out.append((jstar, rem))
    return out


def plan(num_nodes, ids, off, S, start_ids):
    """Changesets from a full cache whose line r holds start_ids[r]."""
    n = len(ids)
    it = np.repeat(np.arange(S), np.diff(off))
    prev, nxt = np.full(n, -2), np.full(n, S)      # -2: no stay leads here, -1: from the start state
    before, first = {}, {}
    for p, v in enumerate(ids):
        if v in before:
            prev[p] = it[before[v]]
            nxt[before[v]] = it[p]
        else:
            first[int(v)] = int(it[p])
        before[v] = p
    line = {int(v): r for r, v in enumerate(start_ids)}
    for v, f in first.items():
        if v in line:
            p = off[f] + int(np.nonzero(ids[off[f]:off[f + 1]] == v)[0][0])
            prev[p] = -1
    start_keys = np.array([first.get(int(v), S) for v in start_ids], dtype=np.int64)
    cut = thresholds(off, nxt, S, start_keys)
    decided = {}                                    # t -> (class that is selected from, id limit)
    bypassed = set()                                # (v, t): incoming rows that the cut of t dropped

    def dropped(i, j, v, until):
        """First t < min(until, j) at which the stay [i, j) of row v ends, else None."""
        for t in range(max(i, 0), min(until, j)):
            if cut[t][0] < j:
                return t
            if cut[t][0] == j and cut[t][1] > 0:
                cls, T = decided[t]
                if (i == t and (v, t) in bypassed) or (cls == "res" and v > T):
                    return t
        return None

    def hit(p):
        return prev[p] != -2 and dropped(prev[p], it[p], int(ids[p]), it[p]) is None

    def inserted(p):
        i = it[p]
        if hit(p) or nxt[p] > cut[i][0]:
            return False
        return nxt[p] < cut[i][0] or cut[i][1] == 0 or (int(ids[p]), i) not in bypassed

    for t in range(S):
        j, rem = cut[t]
        if j > S or rem == 0:
            continue
        res, inc = [], []
        if j < S:
            for q in range(off[j], off[j + 1]):
                if prev[q] != -2 and prev[q] < t and dropped(prev[q], j, int(ids[q]), t) is None:
                    res.append(int(ids[q]))
        else:
            for p in range(off[t]):
                v, i = int(ids[p]), it[p]
                if nxt[p] == S and (hit(p) or inserted(p)) and dropped(i, S, v, t) is None:
                    res.append(v)
            for v, k in zip(start_ids, start_keys):
                if k == S and dropped(-1, S, int(v), t) is None:
                    res.append(int(v))
        for p in range(off[t], off[t + 1]):
            if nxt[p] == j:
                (res if hit(p) else inc).append(int(ids[p]))
        if rem < len(inc):
            decided[t] = ("in", sorted(inc)[len(inc) - rem - 1])
            bypassed |= {(v, t) for v in inc if v > decided[t][1]}
        else:
            bypassed |= {(v, t) for v in inc}
            go = rem - len(inc)
            decided[t] = ("res", sorted(res)[len(res) - go - 1]) if go else ("none", 0)

    # stays from insertion (or the start state) to eviction, then the lines, iteration by iteration
    hits = np.array([hit(p) for p in range(n)], dtype=bool)
    ins = np.array([inserted(p) for p in range(n)], dtype=bool)
    leaves = [[] for _ in range(S + 1)]             # t -> rows evicted by iteration t
    for v, k in zip(start_ids, start_keys):
        t = dropped(-1, int(k), int(v), S)
        if t is not None:
            leaves[t].append(int(v))
    for p in range(n):
        if hits[p] or ins[p]:
            t = dropped(it[p], nxt[p], int(ids[p]), S)
            if t is not None:
                leaves[t].append(int(ids[p]))
    res = {"in_ids": [], "out_ids": [], "in_positions": [], "cs_offsets": [0],
           "miss_count": [], "src_line": np.full(n, -1)}
    for t in range(S):
        at = np.arange(off[t], off[t + 1])
        res["src_line"][at[hits[at]]] = [line[int(v)] for v in ids[at[hits[at]]]]
        out = sorted(leaves[t], key=lambda v: line[v])
        new = at[ins[at]]
        assert len(out) == len(new)
        lines = [line.pop(v) for v in out]
        for p, l in zip(new, lines):
            line[int(ids[p])] = l
        res["in_ids"] += [int(v) for v in ids[new]]
        res["in_positions"] += [int(p - off[t]) for p in new]
        res["out_ids"] += out
        res["cs_offsets"].append(len(res["in_ids"]))
        res["miss_count"].append(int((~hits[at]).sum()))
    return res, cut


def random_trace(rng, hot):
    n = int(rng.integers(2, 90))
    S = int(rng.integers(1, 16))
    weight = rng.random(n) ** (4 if hot else 1) + 1e-9
    tr = [rng.choice(n, size=int(rng.integers(0, min(int(rng.integers(1, 60)), n) + 1)), replace=False,
                     p=weight / weight.sum()) for _ in range(S)]
    off = np.cumsum([0] + [len(x) for x in tr])
    return n, S, np.concatenate(tr).astype(np.int32), off.astype(np.int64)


@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("resumed", [False, True])
def test_changesets_follow_from_stays_and_cuts(hot, resumed):
    rng = np.random.default_rng(11 + 2 * hot + resumed)
    cuts = 0
    for trial in range(150):
        n, S, ids, off = random_trace(rng, hot)
        if resumed:
            cap = int(rng.integers(1, n + 1))
            start = rng.choice(n, size=cap, replace=False).astype(np.int32)
            want = oracle.changeset_resume(n, ids, off, cap, start)
        else:
            distinct = len(np.unique(ids))
            if distinct < 2:
                continue
            cap = int(rng.integers(1, distinct))
            want = oracle.changeset(n, ids, off, cap)
            start = want["init_ids"]
        got, cut = plan(n, ids, off, S, start)
        cuts += sum(1 for j, rem in cut if j <= S and rem)
        for name in ("in_ids", "out_ids", "in_positions", "cs_offsets", "miss_count"):
            assert np.array_equal(np.asarray(got[name]), want[name]), (trial, name)
        lines = oracle.resolve_lines(n, ids, off, start, want["in_ids"], want["out_ids"],
                                     want["cs_offsets"])
        assert np.array_equal(got["src_line"], lines), trial
    assert cuts > 100
