"""Lone patterns: vertices whose loads lie about the even split of one pattern,
below every other's, beside hubs (codes of either width), against the oracle."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import paper_2504_10937_amd as lds
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [3, 4])
@pytest.mark.parametrize("hub", [0, 40])
def test_lone_patterns(mode, hub):
    """3,000 cliques of `mode` vertices on shuffled ids (past the graphs that
    one workgroup runs), alone and beside K_40"""
    announce("lone patterns", mode, hub)
    a, b = np.triu_indices(mode, 1)
    base = (np.arange(3000) * mode)[:, None]
    c, d = np.triu_indices(hub, 1)
    n = 3000 * mode + hub
    ids = np.random.default_rng(mode).permutation(n).astype(np.int32)
    u = np.concatenate([(a + base).ravel(), c + 3000 * mode])
    v = np.concatenate([(b + base).ravel(), d + 3000 * mode])
    for iters in (1, 2, 40):
        check_fw(n, ids[u], ids[v], mode, iters)
