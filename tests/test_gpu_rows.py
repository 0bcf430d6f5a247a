"""Peeling over frontiers that mix rows about the length from which a row is
walked by itself (128 slots) with shorter ones and none, with one vertex a wave
and up to 64, in the one-workgroup tail and over a grid; core and tr-core
numbers as the oracle's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


def _fans(degrees, seed):
    """hubs of the given degrees on leaves of their own, leaves 2i and 2i + 1
    joined (a triangle with the hub), ids shuffled"""
    u, v, n = [], [], 0
    for d in degrees:
        leaf = n + 1 + np.arange(d)
        u += [np.full(d, n), leaf[:-1:2]]
        v += [leaf, leaf[1::2]]
        n += d + 1
    ids = np.random.default_rng(seed).permutation(n).astype(np.int32)
    return n, ids[np.concatenate(u)], ids[np.concatenate(v)]


def _cliques(sizes, seed):
    u, v, n = [], [], 0
    for k in sizes:
        a, b = np.triu_indices(k, 1)
        u.append(a + n)
        v.append(b + n)
        n += k
    ids = np.random.default_rng(seed).permutation(n).astype(np.int32)
    return n, ids[np.concatenate(u)], ids[np.concatenate(v)]


GRAPHS = {
    "fans": lambda: _fans([1, 2, 3, 125, 126, 127, 128, 129, 130, 255, 256, 257, 600], 1),
    "many fans": lambda: _fans([2 + i % 140 for i in range(300)], 2),
    "cliques": lambda: _cliques([2, 3, 16, 17, 63, 64, 65, 127, 128, 129, 130, 150], 3),
    "triangle rows": lambda: _cliques([3, 4, 16, 17, 18, 19, 24, 17, 18], 6),  # 120 and 136 slots a row about 128
    "one clique": lambda: _cliques([1100], 4),
    "path": lambda: (3000, np.arange(2999, dtype=np.int32), np.arange(1, 3000, dtype=np.int32)),
    "many cliques": lambda: _cliques([3 + i % 9 for i in range(2200)], 5),
}


@pytest.mark.parametrize("wg", [None, 2, 9])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_mixed_rows(name, wg, monkeypatch):
    announce("mixed rows", name, wg)
    if wg:
        monkeypatch.setenv("LDS_PEEL_WG", str(wg))
    n, u, v = GRAPHS[name]()
    G = oracle.Graph(n, u, v)
    g = lds.lds_create_graph(n, u, v)
    np.testing.assert_array_equal(lds.lds_core_numbers(g, 2), oracle.core_numbers(G, 2))
    if "clique" not in name or name == "many cliques":
        np.testing.assert_array_equal(lds.lds_core_numbers(g, 3), oracle.core_numbers(G, 3))
