"""The Frank-Wolfe sweep over every shape its plan can take: chunk targets
from one word to the largest, hub rows in short and long pieces, pulled and
pushed; loads, splits and gap exactly as the oracle's."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime first, as a program that shares tensors with the library loads it)

import oracle
import paper_2504_10937_amd as lds
import synth
from gpu_helpers import announce, check_fw
from test_gpu_fw import _all_hub_graph, _hub_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("push", [False, True])
@pytest.mark.parametrize("chunk", [64, 128, 448, 1024])
def test_edge_plans(chunk, push, monkeypatch):
    announce("edge plan", chunk, push)
    monkeypatch.setenv("LDS_SWEEP_CHUNK", str(chunk))
    monkeypatch.setenv("LDS_PUSH_SLOTS", "0" if push else str(1 << 62))
    for n, u, v in (_hub_graph(8), synth.powerlaw_planted(5_003, 2.2, 9.0, 3, 20, 90, 0.5, seed=21)):
        check_fw(n, u, v, 2, 41)


@pytest.mark.parametrize("push", [False, True])
def test_pushed_hubs_to_stable_groups(push, monkeypatch):
    """Alg. 2 reads the pushed slots' splits from their mirrors"""
    announce("push groups", push)
    monkeypatch.setenv("LDS_PUSH_SLOTS", "0" if push else str(1 << 62))
    for n, u, v in (_hub_graph(9), _all_hub_graph(9)):
        G = oracle.Graph(n, u, v)
        ref = oracle.fw_exact(G, 2, 30, with_gap=False)
        g = lds.lds_create_graph(n, u, v)
        lds.lds_frank_wolfe(g, 2, 30)
        groups, lo, hi = lds.lds_stable_groups(g, 2)
        o_groups, o_lo, o_hi = oracle.extract_sg(G, 2, ref["A"], ref["split"], ref["D"])
        assert groups == o_groups
        np.testing.assert_array_equal(lo, o_lo)
        np.testing.assert_array_equal(hi, o_hi)


@pytest.mark.parametrize("chunk", [64, 192, 1024])
def test_triangle_plans(chunk, monkeypatch):
    """hub rows of triangles (rows of more than 1024 slots) in pieces of 512"""
    announce("triangle plan", chunk)
    monkeypatch.setenv("LDS_SWEEP_CHUNK", str(chunk))
    n, u, v = synth.holme_kim(4_001, 12, 0.8, seed=22)
    check_fw(n, u, v, 3, 40)


def test_long_pieces():
    """a plan large enough for the 2048-slot pieces and several rounds of
    chunks per wave (5M slots)"""
    announce("long pieces")
    n, u, v = synth.powerlaw_planted(150_000, 2.1, 24.0, 8, 200, 900, 0.4, seed=23)
    G = oracle.Graph(n, u, v)
    assert 2 * G.m >= 1 << 22
    ref = oracle.fw_exact(G, 2, 6, with_gap=True)
    g = lds.lds_create_graph(n, u, v)
    out = lds.lds_frank_wolfe(g, 2, 6, want_num=True, want_gap=True)
    np.testing.assert_array_equal(out["num"], ref["A"])
    np.testing.assert_allclose(out["gap"], ref["gap"], rtol=1e-12, atol=1e-12 * float(np.abs(ref["gap"]).max()))


def _cycle(n):
    a = np.arange(n, dtype=np.int32)
    return n, a, ((a + 1) % n).astype(np.int32)


def _clique(n):
    u, v = np.triu_indices(n, 1)
    return n, u.astype(np.int32), v.astype(np.int32)


ONE = {
    "pair": lambda: (2, np.array([0], np.int32), np.array([1], np.int32)),
    "star": lambda: (1100, np.zeros(1099, np.int32), np.arange(1, 1100, dtype=np.int32)),
    "k24": lambda: _clique(24),          # triangles: 6072 slots
    "k90": lambda: _clique(90),
    "cycle_8192": lambda: _cycle(8192),  # 16,384 slots: the largest for one workgroup
    "cycle_8193": lambda: _cycle(8193),
    "sparse": lambda: synth.powerlaw_planted(700, 2.3, 6.0, 2, 10, 20, 0.5, seed=31),
}


@pytest.mark.parametrize("mode", [2, 3])
@pytest.mark.parametrize("name", sorted(ONE))
def test_small_graphs_in_one_launch(name, mode):
    announce("one launch", name, mode)
    n, u, v = ONE[name]()
    for iters in (1, 2, 33):
        check_fw(n, u, v, mode, iters)


@pytest.mark.parametrize("threads,lds_vertices", [(256, 8192), (1024, 8192), (512, 0)])
def test_batch_of_word_runs(threads, lds_vertices):
    """hub rows of triangles, keys in memory (n > 8192), more words than LDS
    holds, plans of one word: loads as the oracle's"""
    announce("batch words", threads, lds_vertices)
    graphs = [_clique(50), _clique(3), ONE["star"](), _cycle(9001),
              synth.powerlaw_planted(8_000, 2.2, 40.0, 4, 100, 300, 0.5, seed=32)]
    hs, modes, want, iters = [], [], [], []
    for n, u, v in graphs:
        G = oracle.Graph(n, u, v)
        for mode in (2, 3):
            hs.append(lds.lds_create_graph(n, u, v))
            modes.append(mode)
            iters.append(17)
            want.append(oracle.fw_exact(G, mode, 17, with_gap=False)["A"])
    b = lds.lds_batch_create(hs, modes, iters,
                             tune=lds.lds_tune_default(threads=threads, lds_vertices=lds_vertices,
                                                       max_kernel_cost=1 << 30))
    assert lds.lds_batch_info(b)["kernel_graphs"] == len(hs)
    for _ in range(3):
        lds.lds_batch_run(b)
        for h, m, a in zip(hs, modes, want):
            np.testing.assert_array_equal(lds.lds_loads(h, m, want_num=True)["num"], a)


@pytest.mark.parametrize("leaves", [65_533, 65_534, 65_535, 80_000])
def test_load_codes(leaves):
    """the two widths of the 16-bit load codes, at the largest degree that
    parts them, with loads from 0 to half that degree"""
    announce("load codes", leaves)
    hub = np.zeros(leaves, np.int32)
    leaf = np.arange(3, 3 + leaves, dtype=np.int32)
    u = np.concatenate([[0, 1], hub, hub[: leaves // 2] + 1, leaf[:-1:7]]).astype(np.int32)
    v = np.concatenate([[1, 2], leaf, leaf[: leaves // 2], leaf[1::7][: len(leaf[:-1:7])]]).astype(np.int32)
    check_fw(leaves + 5, u, v, 2, 23)
