"""Core numbers over frontiers of tens of thousands of vertices, exactly as the
oracle's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
import synth
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wg", [2, 16])
@pytest.mark.parametrize("mode", [2, 3])
def test_long_frontiers(mode, wg, monkeypatch):
    """One level peels tens of thousands of vertices: frontiers dealt 64
    vertices to a wave, pushed through LDS and, with two workgroups, past its
    buffer; then an induced subgraph."""
    announce("long frontiers", mode, wg)
    monkeypatch.setenv("LDS_PEEL_WG", str(wg))
    n, u, v = synth.holme_kim(60_000, 4, 0.5, seed=17)
    G = oracle.Graph(n, u, v)
    g = lds.lds_create_graph(n, u, v)
    np.testing.assert_array_equal(lds.lds_core_numbers(g, mode), oracle.core_numbers(G, mode))
    alive = np.random.default_rng(3).random(n) < 0.8
    got = lds.lds_core_numbers(g, mode, alive=alive)
    keep = alive[u] & alive[v]
    H = oracle.Graph(n, u[keep], v[keep])
    np.testing.assert_array_equal(got, np.where(alive, oracle.core_numbers(H, mode), -1))
    g.destroy()
