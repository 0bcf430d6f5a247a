"""Ingest of graphs with buckets of rows past a workgroup's LDS (24,576 keys):
rows of large degree alone, several to a bucket and in several buckets, pairs
given very often, ids that agree in their low bits; refusals in strict mode.
Degrees and rows are checked through the oracle's exact Frank-Wolfe results and
core numbers."""
import numpy as np
import pytest
import torch

import oracle
import paper_2504_10937_amd as lds
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


def _pairs(n, pairs, seed):
    rng = np.random.default_rng(seed)
    return rng.integers(0, n, pairs).astype(np.int32), rng.integers(0, n, pairs).astype(np.int32)


def _hubs(n, ids, leaves, pairs, seed):
    """`leaves` distinct neighbours for each of the hubs, on a random graph"""
    rng = np.random.default_rng(seed)
    u, v = _pairs(n, pairs, seed)
    nb = [rng.permutation(n)[:leaves].astype(np.int32) for _ in ids]
    return n, np.concatenate([u] + [np.full(leaves, h, np.int32) for h in ids]), np.concatenate([v] + nb)


def _star(n, hub, leaves):
    """a row of `leaves` keys alone in its bucket"""
    ids = np.arange(n, dtype=np.int32)
    nb = ids[(ids & 255) != (hub & 255)][:leaves]
    return n, np.full(leaves, hub, np.int32), nb


def _copies(n, pairs, copies, seed):
    u, v = _pairs(n, pairs, seed)
    a = np.full(copies, 3, np.int32)
    return n, np.concatenate([u, a, a + 1]), np.concatenate([v, a + 1, a])


CASES = {
    "keys_24576": lambda: _star(100_000, 7, 24_576),  # the last bucket that fits, and the first that does not
    "keys_24577": lambda: _star(100_000, 7, 24_577),
    "one_hub": lambda: _hubs(150_000, [149_999], 140_000, 200_000, 3),
    "hubs_apart": lambda: _hubs(60_000, [0, 5, 77, 4_001, 59_999], 30_000, 100_000, 4),
    "hubs_together": lambda: _hubs(70_000, [64 * 1_024, 0, 32 * 1_024, 1_024], 25_000, 50_000, 5),
    "copies": lambda: _copies(50_000, 300_000, 60_000, 6),       # 120,000 keys, two slots
    "one_bucket": lambda: (1 << 22, *(x * 16_384 for x in _pairs(256, 100_000, 7))),
    "few_buckets": lambda: (1 << 22, *(x * 512 for x in _pairs(8_192, 400_000, 8))),
}


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_overfull_buckets(name, device):
    announce("overfull", name, device)
    n, u, v = CASES[name]()
    G = oracle.Graph(n, u, v)
    args = (torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()) if device else (u, v)
    g = lds.lds_create_graph(n, *args)
    assert lds.lds_graph_info(g)["m"] == G.m
    check_fw(n, u, v, 2, 3, G=G, gpu_graph=g)
    np.testing.assert_array_equal(lds.lds_core_numbers(g, 2), oracle.core_numbers(G, 2))


def test_strict():
    announce("overfull strict")
    n, h = 200_000, 30_000
    u, v = np.zeros(h, np.int32), np.arange(1, h + 1, dtype=np.int32)
    assert lds.lds_graph_info(lds.lds_create_graph(n, u, v, flags=lds.LDS_STRICT))["m"] == h
    for x, y in ((0, 0), (h, 0), (0, h), (0, n)):  # a loop, copies in either order, an id out of range
        with pytest.raises(lds.LdsError) as e:
            lds.lds_create_graph(n, np.append(u, x).astype(np.int32), np.append(v, y).astype(np.int32),
                                 flags=lds.LDS_STRICT)
        assert e.value.status == 1
