"""Graphs on either side of what one workgroup runs in one launch (12,288 slots,
each four vertices counting as one), against the oracle."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import paper_2504_10937_amd as lds  # noqa: F401
from gpu_helpers import announce, check_fw

pytestmark = pytest.mark.gpu


def _cycle(n):
    a = np.arange(n, dtype=np.int32)
    return n, a, ((a + 1) % n).astype(np.int32)


def _clique(k, pendants):
    """K_k and pendant vertices, which have no triangle"""
    u, v = np.triu_indices(k, 1)
    p = np.arange(pendants)
    return k + pendants, np.append(u, p % k).astype(np.int32), np.append(v, k + p).astype(np.int32)


@pytest.mark.parametrize("mode,graph", [(2, (_cycle, 5461)), (2, (_cycle, 5462)), (3, (_clique, 30, 402)),
                                        (3, (_clique, 30, 406)), (2, (_clique, 111, 0)), (2, (_clique, 112, 0))])
def test_either_side(mode, graph):
    announce("one workgroup or sweeps", mode, graph[1:])
    for iters in (1, 2, 33):
        check_fw(*graph[0](*graph[1:]), mode, iters)
