"""Hub rows in pieces of 512, 1024 and 2048 slots (few and many hub slots, plans
on either side of 2^22 slots), rows that end within a piece, all modes; loads,
splits and gap as the oracle's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import paper_2504_10937_amd as lds
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


def _bipartite(a, b):
    u = np.repeat(np.arange(a, dtype=np.int32), b)
    return a + b, u, np.tile(np.arange(a, a + b, dtype=np.int32), a)


def _clique(k):
    u, v = np.triu_indices(k, 1)
    return k, u.astype(np.int32), v.astype(np.int32)


@pytest.mark.parametrize("mode,graph,args,hubs", [
    (2, _bipartite, (3, 5_001), 3), (2, _bipartite, (20, 40_003), 20), (2, _bipartite, (70, 31_000), 70),
    (3, _clique, (70,), 70), (3, _clique, (125,), 125), (4, _clique, (30,), 30), (4, _clique, (50,), 50)])
def test_pieces(mode, graph, args, hubs):
    announce("pieces", mode, args)
    g = check_fw(*graph(*args), mode, 6)[0]
    assert lds.lds_sweep_info(g, mode)["hub_rows"] == hubs
