"""Batches of triangle and 4-clique slots, and 4-clique slots of three 21-bit
ids (plans up to 2^21 vertices) and of three 32-bit ids (above): for these,
small components of cliques at the far end of the internal ids, next to a
clique-free graph of larger degree that fills the ids below them.  Their
loads, splits and gap equal those of the components alone, which the oracle
checks."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import paper_2504_10937_amd as lds
import synth
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


def _components():
    """K4, K5 and two K4s sharing an edge (degrees at most 5), 40 of each"""
    shapes = [(4, [(a, b) for a in range(4) for b in range(a)]), (5, [(a, b) for a in range(5) for b in range(a)]),
              (6, sorted({(a, b) for q in ((0, 1, 2, 3), (0, 1, 4, 5)) for a in q for b in q if b < a}))]
    u, v, n = [], [], 0
    for i in range(120):
        k, e = shapes[i % 3]
        u += [n + a for a, _ in e]
        v += [n + b for _, b in e]
        n += k
    return n, np.array(u, np.int32), np.array(v, np.int32)


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1])
def test_packed_edge(n):
    announce("packed slots", n)
    k, u, v = _components()
    _, _, ref, _ = check_fw(k, u, v, 4, 17)
    small = lds.lds_create_graph(k, u, v)
    lds.lds_frank_wolfe(small, 4, 17)
    sv, sn = lds.lds_splits(small, 4)
    # degree 6, no triangle: ids i, i + 1, i + 3, i + 9 around a ring
    f = n - k
    i = np.arange(f, dtype=np.int64)
    fu = np.concatenate([i, i, i])
    fv = np.concatenate([(i + d) % f for d in (1, 3, 9)])
    g = lds.lds_create_graph(n, np.concatenate([fu, u.astype(np.int64) + f]).astype(np.int32),
                             np.concatenate([fv, v.astype(np.int64) + f]).astype(np.int32))
    out = lds.lds_frank_wolfe(g, 4, 17, want_num=True, want_gap=True)
    np.testing.assert_array_equal(out["num"][f:], ref["num"])
    assert not out["num"][:f].any()
    np.testing.assert_array_equal(out["gap"], ref["gap"])
    bv, bn = lds.lds_splits(g, 4)
    np.testing.assert_array_equal(bv, sv + f)
    np.testing.assert_array_equal(bn, sn)


def _dense(k, seed):
    """K_k without a few edges, some of its vertices tied to a sparse tail"""
    rng = np.random.default_rng(seed)
    u, v = np.triu_indices(k, 1)
    keep = rng.random(len(u)) > 0.02
    n, s, d = synth.holme_kim(2_000, 6, 0.8, seed=seed)
    a, b = rng.integers(0, k, 500), rng.integers(k, k + n, 500)
    return k + n, np.concatenate([u[keep], s + k, a]).astype(np.int32), np.concatenate([v[keep], d + k, b]).astype(np.int32)


@pytest.mark.parametrize("mode,k", [(3, 150), (3, 230), (4, 40), (4, 82)])
def test_batches_of_words(mode, k):
    """fewer and more than 2^22 slots (four and eight words a batch), hub
    pieces and chunks, every code in LDS"""
    n, s, d = _dense(k, seed=k)
    announce("batches of words", mode, k)
    g = check_fw(n, s, d, mode, 7)[0]
    assert (lds.lds_sweep_info(g, mode)["slots"] >= 1 << 22) == (k in (230, 82))


def test_hot_and_cold_codes():
    """more vertices than codes in LDS: batches of either kind and mixed ones"""
    announce("hot and cold codes")
    check_fw(*synth.holme_kim(90_000, 6, 0.7, seed=5), 3, 9)
