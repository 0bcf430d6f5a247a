"""More items than the threads of one launch, or than its single-pass tiles:
sizes at which a kernel takes turns."""
import numpy as np
import pytest
import torch

import paper_2504_10937_amd as lds
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


def test_listing_units_past_one_launch():
    """2^26 units of oriented edges, a wave each, are 2^32 threads: the ring
    i, i + 1, i + 2 has a unit per vertex, n triangles and three at each vertex"""
    n = (1 << 26) + 9
    announce("listing units", n)
    i = torch.arange(n, dtype=torch.int32, device="cuda")
    u = torch.cat([i, i])
    v = torch.cat([(i + 1) % n, (i + 2) % n]).to(torch.int32)
    g = lds.lds_create_graph(n, u, v)
    assert lds.lds_graph_info(g)["m"] == 2 * n
    T, tc = lds.lds_triangles(g, want_list=False, want_counts=True)[0::2]
    assert T == n
    assert tc.shape == (n,) and (tc == 3).all()
    g.destroy()


def test_wide_tiles_with_payload():
    """the order of 2^23 + 77 loads: a sort of keys with ids by the wide tiles,
    the last of them a remainder"""
    n = (1 << 23) + 77
    announce("wide tiles with payload", n)
    gen = torch.Generator(device="cuda").manual_seed(9)
    u = torch.randint(0, n, (3_000_000,), generator=gen, device="cuda", dtype=torch.int32)
    v = torch.randint(0, n // 50, (3_000_000,), generator=gen, device="cuda", dtype=torch.int32)
    g = lds.lds_create_graph(n, u, v)
    num = lds.lds_frank_wolfe(g, 2, 3, want_num=True)["num"]
    order, E, inI = lds.lds_sort_prefix(g, 2)
    want = np.lexsort((np.arange(n), -num.astype(np.int64)))
    np.testing.assert_array_equal(order, want)
    assert E[-1] == lds.lds_graph_info(g)["m"]
    g.destroy()
