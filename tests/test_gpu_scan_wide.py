"""The stable-group scan as for a plan of 2^32 records, whose offsets are read at
full width: groups and bounds as the oracle's, in one workgroup and on a grid."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
import synth
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wg", [1, 7])
@pytest.mark.parametrize("mode,iters", [(2, 60), (3, 40)])
def test_wide_offsets(mode, iters, wg, monkeypatch):
    announce("wide offsets", mode, wg)
    monkeypatch.setenv("LDS_SCAN_WIDE", "1")
    monkeypatch.setenv("LDS_SCAN_WG", str(wg))
    n, u, v = synth.powerlaw_planted(4_000, 2.3, 9.0, 6, 20, 60, 0.5, seed=41)
    G = oracle.Graph(n, u, v)
    ref = oracle.fw_exact(G, mode, iters, with_gap=False)
    g = lds.lds_create_graph(n, u, v)
    lds.lds_frank_wolfe(g, mode, iters)
    groups, lo, hi = lds.lds_stable_groups(g, mode)
    o_groups, o_lo, o_hi = oracle.extract_sg(G, mode, ref["A"], ref["split"], ref["D"])
    assert groups == o_groups
    np.testing.assert_array_equal(lo, o_lo)
    np.testing.assert_array_equal(hi, o_hi)
