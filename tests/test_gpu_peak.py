"""Device memory that ingest takes at its peak, from host arrays: 20 bytes a key
(two keys a pair) on either route, the copies of the arrays being given back
once the keys are made, beside the radix counters (a quarter byte a key) and
arrays by vertex."""
import gc

import numpy as np
import pytest
import torch

import paper_2504_10937_amd as lds
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,n", [("buckets", 300_000), ("full sort", 1_000)])
def test_ingest_peak(name, n):
    announce("ingest peak", name)
    rng = np.random.default_rng(n)
    pairs = 8_000_000
    u = rng.integers(0, n, pairs).astype(np.int32)
    v = rng.integers(0, n, pairs).astype(np.int32)
    gc.collect()
    lds.lds_set_allocator(True)
    try:
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        torch.cuda.reset_peak_memory_stats()
        g = lds.lds_create_graph(n, u, v)
        peak = torch.cuda.max_memory_allocated() - before
        g.destroy()
    finally:
        gc.collect()
        lds.lds_set_allocator(False)
    assert peak <= 20.5 * 2 * pairs + 64 * n + (4 << 20)
