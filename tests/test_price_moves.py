"""The search of the price solve moves tokens along shortest paths and relabels their listed exchanges instead of reading their rows again.  A
model of that on the CPU, against exchanges rebuilt from the rows: the relabelled ones have the reduced costs of where the token is now,
and what the list lacks of a moved token costs at least the bound less what its moves cost.  (No GPU.)"""
import numpy as np
import pytest


@pytest.mark.parametrize("seed", range(12))
def test_relabelled_exchanges(seed):
    rng = np.random.default_rng(seed)
    T, E, k, B = int(rng.integers(6, 40)), int(rng.integers(4, 12)), int(rng.integers(1, 4)), int(rng.integers(20, 120))
    q = rng.integers(0, 200, (T, E))
    p = rng.integers(0, 60, E)
    held = [set(int(e) for e in np.argsort(-(q[u] - p), kind="stable")[:k]) for u in range(T)]
    value = lambda u, e: int(q[u, e] - p[e])
    arcs = [[u, a, b, value(u, a) - value(u, b)] for u in range(T) for a in held[u] for b in range(E)
            if b not in held[u] and value(u, a) - value(u, b) < B]          # token, from, to, reduced cost
    pi = np.zeros(E, np.int64)
    cost = np.zeros(T, np.int64)                                            # of a token's moves, at the prices of the start
    moves = 0
    for search in range(10):
        root, target = (int(x) for x in rng.choice(E, 2, replace=False))
        dist, last = {root: 0}, {}
        for _ in range(E):                                                  # Bellman-Ford
            for i, (u, a, b, c) in enumerate(arcs):
                if a in dist and dist[a] + c < dist.get(b, 1 << 40):
                    dist[b], last[b] = dist[a] + c, i
        if target not in dist:
            continue
        path, at = [], target
        while at != root:
            path.append(last[at])
            at = arcs[last[at]][1]
        add = np.array([min(dist.get(e, 1 << 40), dist[target]) for e in range(E)])
        pi += add
        moved = {}
        for i in path:
            u, a, b, _ = arcs[i]
            moved.setdefault(u, []).append((a, b))
        for arc in arcs:
            u, a, b, c = arc
            arc[3] = c + int(add[a] - add[b])
            for x, y in moved.get(u, ()):                                   # the places of several moves of a token are all different
                if a == x:
                    arc[1] = y
                if b == y:
                    arc[2] = x
        for u, m in moved.items():
            assert len({e for xy in m for e in xy}) == 2 * len(m)
            for x, y in m:
                held[u].remove(x)
                held[u].add(y)
                cost[u] += max(0, int(pi[y] - pi[x]))
                moves += 1
        listed = {}
        for u, a, b, c in arcs:
            assert a in held[u] and b not in held[u] and c == value(u, a) + pi[a] - value(u, b) - pi[b] and c >= 0
            listed[u, a, b] = c
        apart = int(pi.max() - pi.min())
        for u in range(T):
            for a in held[u]:
                for b in range(E):
                    if b not in held[u] and (u, a, b) not in listed:
                        assert value(u, a) + pi[a] - value(u, b) - pi[b] >= B - cost[u] - apart
    assert moves > 0 or len(arcs) < E
