"""lds_fw_elapsed counts sweeps, one per iteration, whether they are launches of
their own or all in one."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import paper_2504_10937_amd as lds
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pairs,iters", [(50, 200, 37), (20_000, 60_000, 37), (50, 0, 5)])
def test_sweeps(n, pairs, iters):
    announce("elapsed", n, pairs)
    rng = np.random.default_rng(n)
    g = lds.lds_create_graph(n, rng.integers(0, n, pairs).astype(np.int32), rng.integers(0, n, pairs).astype(np.int32))
    lds.lds_frank_wolfe(g, 2, iters)
    ms, sweeps = lds.lds_fw_elapsed(g, 2)
    assert ms >= 0 and sweeps == (iters if pairs else 0)
