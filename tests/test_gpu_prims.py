"""Scans, sorts and suffix maxima at the edges of their tiles, through the
calls that use them: ingest (sort of 2 keys per pair, scans over vertices),
the order of the loads, prefix counts and the candidate set."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pairs", [(3, 1), (63, 64), (500, 2047), (500, 2048), (500, 2049), (4096, 6000),
                                     (4097, 2048), (12288, 9000), (12289, 9001), (16385, 20000), (70001, 90000)])
def test_tile_edges(n, pairs):
    announce("tile edges", n, pairs)
    rng = np.random.default_rng(n + pairs)
    # endpoints crowd on the small ids: duplicates, loops, long and empty rows
    u = (n * rng.random(pairs) ** 2).astype(np.int32)
    v = rng.integers(0, n, pairs).astype(np.int32)
    G = oracle.Graph(n, u, v)
    g = lds.lds_create_graph(n, u, v)
    assert lds.lds_graph_info(g)["m"] == G.m
    check_fw(n, u, v, 2, 9, G=G, gpu_graph=g)
    ref = oracle.fw_exact(G, 2, 9, with_gap=False)
    order, E, inI = lds.lds_sort_prefix(g, 2)
    o_order, o_E, o_inI = oracle.sort_prefix(G, 2, ref["A"])
    np.testing.assert_array_equal(order, o_order)
    np.testing.assert_array_equal(E, o_E)
    np.testing.assert_array_equal(inI, o_inI)
