"""Triangle and 4-clique listing at the edges of its work units: out-lists
around the 64 edges of a unit, longer than the 1024 entries staged per wave,
walked and probed, and per-vertex counts past the histogram's ids; exactly
against the oracle."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
import synth
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


def clique(n):
    u, v = np.triu_indices(n, 1)
    return n, u.astype(np.int32), v.astype(np.int32)


def wide_lists(na, nb):
    """nb vertices joined to all of a ring of na vertices of larger degree:
    out-lists of na entries, one triangle per ring edge and vertex."""
    a = np.arange(na)
    bu, bv = np.meshgrid(np.arange(na, na + nb), a, indexing="ij")
    u = np.concatenate([a, bu.ravel()])
    v = np.concatenate([(a + 1) % na, bv.ravel()])
    return na + nb, u.astype(np.int32), v.astype(np.int32)


def far_block():
    """50,000 disjoint triangles: most members' ids lie past the count
    histogram"""
    n = 150_000
    t = np.arange(0, n, 3)
    u = np.concatenate([t, t, t + 1])
    v = np.concatenate([t + 1, t + 2, t + 2])
    return n, u.astype(np.int32), v.astype(np.int32)


CASES = {
    "edgeless": lambda: (7, np.empty(0, np.int32), np.empty(0, np.int32)),
    "one_edge": lambda: (2, np.array([0], np.int32), np.array([1], np.int32)),
    "k3": lambda: clique(3),
    "k65": lambda: clique(65),
    "k66": lambda: clique(66),
    "k130": lambda: clique(130),
    "list_1024": lambda: wide_lists(1024, 1030),
    "list_1025": lambda: wide_lists(1025, 1031),
    "list_1100": lambda: wide_lists(1100, 1200),
    "far": far_block,
    "powerlaw": lambda: synth.powerlaw_planted(20_000, 2.1, 14.0, 5, 30, 200, 0.4, seed=11),
    "attachment": lambda: synth.holme_kim(3_001, 9, 0.7, seed=12),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_triangles(name):
    announce("listing", name)
    n, u, v = CASES[name]()
    G = oracle.Graph(n, u, v)
    want = np.asarray(oracle.triangles(G)[0]).reshape(-1, 3)
    want = np.sort(want, axis=1)
    want = want[np.lexsort(want.T[::-1])]
    T, tri, cnt = lds.lds_triangles(lds.lds_create_graph(n, u, v), want_list=True, want_counts=True)
    assert T == len(want)
    np.testing.assert_array_equal(tri, want)
    np.testing.assert_array_equal(cnt, np.bincount(want.ravel(), minlength=n))


@pytest.mark.parametrize("name", ["k3", "k66", "attachment"])
def test_cliques(name):
    announce("cliques", name)
    n, u, v = CASES[name]()
    Q, q, cnt = lds.lds_cliques4(lds.lds_create_graph(n, u, v), want_list=True, want_counts=True)
    adj = [set() for _ in range(n)]
    for a, b in zip(u.tolist(), v.tolist()):
        if a != b:
            adj[a].add(b)
            adj[b].add(a)
    want = 0
    per = np.zeros(n, np.int64)
    for a, b, c in np.sort(np.asarray(oracle.triangles(oracle.Graph(n, u, v))[0]).reshape(-1, 3), axis=1).tolist():
        for d in adj[a] & adj[b] & adj[c]:
            if d > c:
                want += 1
                per[[a, b, c, d]] += 1
    assert Q == want
    np.testing.assert_array_equal(cnt, per)
    np.testing.assert_array_equal(np.bincount(q.ravel(), minlength=n), per)


@pytest.mark.parametrize("joined", [1, 3])
@pytest.mark.parametrize("hubs", [5, 16, 17, 21, 22, 90])
def test_clique_candidates(hubs, joined):
    """a triangle (a, b, c) whose edge (a, b) has few or many further
    triangles, against the few hubs that c is joined to"""
    announce("clique candidates", hubs, joined)
    a, b, c, leaf = 0, 1, 2, 3 + hubs
    e = [(a, b), (a, c), (b, c)]
    for h in range(3, 3 + hubs):
        e += [(a, h), (b, h)]
        e += [(h, leaf + i) for i in range(250)]
        leaf += 250
    e += [(c, 3 + h) for h in range(0, hubs, max(1, hubs // joined))][:joined]
    e += [(c, leaf + i) for i in range(150)]
    u, v = np.array(e, np.int32).T
    n = leaf + 150
    Q, q, _ = lds.lds_cliques4(lds.lds_create_graph(n, u, v), want_list=True, want_counts=True)
    want, _ = oracle.cliques4(oracle.Graph(n, u, v))
    assert Q == len(want) == joined
    np.testing.assert_array_equal(q, want)
