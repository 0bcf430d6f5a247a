"""Ingest on every route: one-workgroup sort, buckets of rows (small, large and
overflowing ones, one and two passes), full sort; duplicates, loops, crowded
and sparse ids; refusals in strict mode.  Degrees and rows are checked through
the triangle-free and exact Frank-Wolfe results of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2504_10937_amd as lds
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


def random_pairs(n, pairs, seed, crowd=1.0):
    rng = np.random.default_rng(seed)
    return n, (n * rng.random(pairs) ** crowd).astype(np.int32), rng.integers(0, n, pairs).astype(np.int32)


def star(leaves, extra, seed):
    n, u, v = random_pairs(leaves + 1, extra, seed)
    return n, np.concatenate([np.zeros(leaves, np.int32), u]), np.concatenate(
        [np.arange(1, leaves + 1, dtype=np.int32), v])


def hubs(count, leaves, step, extra, seed):
    """`count` hubs whose ids agree in their low bits, with copies and loops"""
    n, u, v = random_pairs(count * step * 64 + leaves, extra, seed)
    h = np.repeat(np.arange(count, dtype=np.int32) * (step * 64), leaves)
    w = np.tile(np.arange(leaves, dtype=np.int32), count)
    return n, np.concatenate([h, u, h[:500]]), np.concatenate([w, v, w[:500]])


CASES = {
    "buckets_2": lambda: random_pairs(700, 2_049, 1),
    "rows_below_buckets": lambda: random_pairs(40, 50_000, 2),     # mostly duplicates, tiny n
    "one_pass": lambda: random_pairs(5_000, 60_000, 3),
    "two_passes": lambda: random_pairs(60_000, 400_000, 4),
    "large_bucket": lambda: star(9_000, 30_000, 5),                # a row of 9000 keys
    "largest_bucket": lambda: star(24_000, 200, 6),
    "grouped_buckets": lambda: hubs(9, 9_000, 64, 20_000, 10),     # hubs that share one bucket, three groups
    "grouped_by_one": lambda: hubs(3, 24_000, 64, 3_000, 11),      # a row a group
    "overflowing_bucket": lambda: star(60_000, 20_000, 7),         # full sort
    "crowded": lambda: random_pairs(1_000_000, 150_000, 8, crowd=6.0),
    "sparse": lambda: random_pairs(3_000_000, 5_000, 9),
    "loops_and_copies": lambda: (50, np.tile(np.arange(50, dtype=np.int32), 200),
                                 np.repeat(np.arange(50, dtype=np.int32), 200)),
}


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_routes(name, device):
    announce("ingest", name, device)
    n, u, v = CASES[name]()
    G = oracle.Graph(n, u, v)
    args = (torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda()) if device else (u, v)
    g = lds.lds_create_graph(n, *args)
    assert lds.lds_graph_info(g)["m"] == G.m
    check_fw(n, u, v, 2, 5, G=G, gpu_graph=g)
    np.testing.assert_array_equal(lds.lds_core_numbers(g, 2), oracle.core_numbers(G, 2))


@pytest.mark.parametrize("pairs", [100, 4_000, 300_000])
def test_refusals(pairs):
    announce("ingest refusals", pairs)
    n = 200_000
    a = np.arange(pairs, dtype=np.int32) % (n // 2)
    b = (a + 1 + np.arange(pairs, dtype=np.int32) // (n // 2)).astype(np.int32)
    g = lds.lds_create_graph(n, a, b, flags=lds.LDS_STRICT)  # distinct pairs
    assert lds.lds_graph_info(g)["m"] == pairs
    for change, strict in (((-1, 3), 0), ((3, n), 0), ((7, 7), lds.LDS_STRICT), ((b[0], a[0]), lds.LDS_STRICT)):
        x, y = a.copy(), b.copy()
        x[-1], y[-1] = change
        with pytest.raises(lds.LdsError) as e:
            lds.lds_create_graph(n, x, y, flags=strict)
        assert e.value.status == 1
    x = a.copy()
    x[-1] = b[-1]  # a loop is dropped otherwise
    assert lds.lds_graph_info(lds.lds_create_graph(n, x, b))["m"] == pairs - 1
