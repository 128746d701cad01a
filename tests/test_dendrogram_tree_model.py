"""A host model of the dendrogram that is read off the Borůvka tree, checked against the oracle's union-find pass
(Alg. 1 step 3).

The library gives every component of every Borůvka round a node, with the smallest edge that leaves it. A row belongs
to the chain of the first node at or above the one where its two ends meet whose leaving edge is larger than the row;
in key order a chain's rows are each other's parents, the last one's parent is the leaving edge; a row joins the rows
before it in its chain to the component that chose it, and the first row, chosen from both sides, joins two.

The model runs these steps on the oracle's forests, with rounds on all edges, or split at a pivot (light rounds first,
then rounds on all of them) before any round, and with a cutoff; children, sizes and parents must be the oracle's for
every row. Mistakes planted in the model (the model, not the library) must show. It is a check of the construction:
the kernels are compared with the oracle on the GPU.
"""
import numpy as np
import pytest

import oracle
import synth

INF = 1 << 60


def boruvka_tree(n, tail, head, splits):
    """Nodes 0..n-1 are the records; returns parent, best (smallest row leaving each node, INF if none) and, per row,
    whether each end's side chose it: chooser[row] = list of nodes. splits: {round: fraction} of the live rows (the
    lighter part) that rounds work on alone until none of them is left."""
    m = len(tail)
    parent, best = list(range(n)), [INF] * n
    chooser = [[] for _ in range(m)]

    def top(x):
        while parent[x] != x:
            x = parent[x]
        return x

    live, parked, r = list(range(m)), [], 0
    while True:
        live = [e for e in live if top(tail[e]) != top(head[e])]
        if not live:
            if not parked:
                return parent, best, chooser
            live, parked = parked, []
            continue
        if r in splits and not parked:
            k = int(len(live) * splits[r])
            if 0 < k < len(live):
                live, parked = live[:k], live[k:]  # rows are in key order
        r += 1
        mins = {}
        for e in live:
            for x in (top(tail[e]), top(head[e])):
                mins[x] = min(mins.get(x, INF), e)
        for x, e in mins.items():
            best[x] = e
            chooser[e].append(x)
        # components of the chosen rows become the next nodes
        comp = {x: x for x in mins}

        def find(x):
            while comp[x] != x:
                x = comp[x]
            return x

        for x, e in mins.items():
            a, b = find(top(tail[e])), find(top(head[e]))
            if a != b:
                comp[max(a, b)] = min(a, b)
        new = {}
        for x in sorted(mins):
            root = find(x)
            if root not in new:
                new[root] = len(parent)
                parent.append(len(parent))
                best.append(INF)
        for x in mins:
            parent[x] = new[find(x)]


def model(n, tail, head, splits=(), mistake=None):
    """Children (node ids: record < n, else n + row), size and parent (row or -1) of every row; parent of records."""
    m = len(tail)
    parent, best, chooser = boruvka_tree(n, tail, head, dict(splits))
    chain, second = [None] * m, {}
    for e in range(m):
        x, y = int(tail[e]), int(head[e])
        while x != y:
            if x < y:
                x = parent[x]
            else:
                y = parent[y]
        S = x
        if mistake != "no climb":
            while e > best[S]:
                S = parent[S]
        chain[e] = S
        assert chooser[e]
        if len(chooser[e]) == 2:
            assert S not in second  # one mutual row a chain: its first
            second[S] = chooser[e][1]
    rows = {}
    for e in range(m):
        rows.setdefault(chain[e], []).append(e)
    last = {S: r[-1] for S, r in rows.items()}
    node_of = lambda z: z if z < n else n + last[z]
    left, right, size, par = [0] * m, [0] * m, [0] * m, [-1] * m
    total = {}
    for S in sorted(rows):  # a chooser's node is of an earlier round, so its chain's total is known
        got = 0
        for k, e in enumerate(rows[S]):
            z = chooser[e][0]
            join = 1 if z < n else total[z]
            if k == 0:
                y = second[S]
                a = node_of(y)
                join += 1 if y < n else total[y]
            else:
                a = n + rows[S][k - 1]
            got += join
            left[e], right[e], size[e] = a, node_of(z), got
            if k + 1 < len(rows[S]):
                par[e] = rows[S][k + 1]
            elif best[S] < m:
                par[e] = best[S] if mistake != "top parent" else -1
        total[S] = got
    rec = [best[x] if best[x] < m else -1 for x in range(n)]
    return left, right, size, par, rec


def matches(n, r, splits=(), cut=None, mistake=None):
    """The model on the oracle's forest (its first `cut` rows after the chains are known) gives the oracle's rows."""
    m = r.m
    left, right, size, par, rec = model(n, r.msf_tail, r.msf_head, splits, mistake)
    if cut is not None:
        m = cut
        par = [p if p < cut else -1 for p in par]
        rec = [p if p < cut else -1 for p in rec]
    ok = all(sorted((left[j], right[j])) == [r.sl_left[j], r.sl_right[j]] and size[j] == r.sl_size[j]
             for j in range(m))
    want_par, want_rec = [-1] * m, [-1] * n
    for j in range(m):
        for c in (int(r.sl_left[j]), int(r.sl_right[j])):
            if c < n:
                want_rec[c] = j
            else:
                want_par[c - n] = j
    return ok and par[:m] == want_par and rec == want_rec


def forests():
    rng = np.random.default_rng(5)
    for k in range(40):
        n = int(rng.integers(2, 160))
        V = int(rng.integers(2, 20))
        s = rng.integers(0, V, n).astype(np.int32)
        d = rng.integers(0, V - 1, n).astype(np.int32)
        d[d >= s] += 1
        yield s, d, rng.integers(0, int(rng.choice([3, 50, 10 ** 6])), n).astype(np.int64), V
    for n in (2, 3, 64, 257):  # one vertex: growing, regular, nested gaps
        k = np.arange(n, dtype=np.int64)
        for t in (np.cumsum(k), 60 * k, np.concatenate([[0], np.cumsum((k[1:] & -k[1:]) * 8 + 1)])):
            yield np.zeros(n, np.int32), np.arange(1, n + 1, dtype=np.int32), t, n + 1
    yield (*synth.chung_lu_bursts(600, 40, 3), 40)


@pytest.mark.parametrize("splits", [(), ((1, 0.5),), ((0, 0.3), (3, 0.6)), ((2, 0.1),)])
def test_rows_equal_the_union_find_pass(splits):
    for s, d, t, V in forests():
        r = oracle.cluster(s, d, t, 3, V, tier=1)
        assert r.status == 0
        assert matches(len(s), r, splits)
        assert matches(len(s), r, splits, cut=r.m // 2)


@pytest.mark.parametrize("mistake", ["no climb", "top parent"])
def test_planted_mistakes_show(mistake):
    shown = 0
    for s, d, t, V in forests():
        r = oracle.cluster(s, d, t, 3, V, tier=1)
        try:
            shown += not matches(len(s), r, mistake=mistake)
        except (AssertionError, KeyError):
            shown += 1
    assert shown > 20
