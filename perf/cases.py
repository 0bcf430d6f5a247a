"""The work that users of the library have it do, as timed cases.

Every case builds seeded synthetic inputs of the shapes this repository's
tests and benchmark use (power-law graphs with planted dense blocks,
preferential attachment with and without triad formation) and makes one pass
through the public entry points:

  step     edge list -> graph, Frank-Wolfe with the gap, stable groups
  groups   Frank-Wolfe with the gap and stable groups on a resident graph
  fw       Frank-Wolfe with the gap on a resident graph
  listing  edge list -> graph, triangle listing with the per-vertex counts
  cliques  edge list -> graph, 4-clique listing, Frank-Wolfe over 4-cliques
  topk     one top-k query on a resident graph
  batch    one run of a captured batch of uneven graphs
  cores    core (tr-core) numbers of a resident graph
"""
import math

import numpy as np
import torch

import paper_2504_10937_amd as lds

EDGE, TRIANGLE, CLIQUE4 = 2, 3, 4

_state = {"allocator": False}


def _library():
    """The library with its buffers in torch's caching allocator (once per
    process, before any graph exists), as the benchmark sets it up."""
    if not _state["allocator"]:
        lds.load()
        lds.lds_set_allocator(True)
        _state["allocator"] = True
    return lds


# ------------------------------------------------------------------ inputs
def _generator(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _powerlaw_offset(n, a, pairs):
    """i0 of the weights (i + i0)^-a whose largest expected degree is
    sqrt(2 pairs), the cap of the Chung-Lu model."""
    cap = math.sqrt(2.0 * pairs)
    lo, hi = 1e-3, float(n) + 1.0
    for _ in range(60):
        mid = math.sqrt(lo * hi)
        total = ((n + mid) ** (1.0 - a) - mid ** (1.0 - a)) / (1.0 - a)
        if 2.0 * pairs * mid ** (-a) / total > cap:
            lo = mid
        else:
            hi = mid
    return hi


def _blocks(n, count, s_lo, s_hi, p, gen):
    """Planted G(s, p) blocks on consecutive ids (permuted by the caller)."""
    us, vs = [], []
    base = 0
    sizes = torch.randint(s_lo, s_hi + 1, (count,), generator=gen, device=gen.device).tolist()
    for s in sizes:
        s = min(s, n - base)
        if s < 2:
            break
        hit = torch.triu(torch.rand(s, s, generator=gen, device=gen.device) < p, diagonal=1).nonzero()
        us.append(hit[:, 0] + base)
        vs.append(hit[:, 1] + base)
        base += s
    return us, vs


def _powerlaw(case, seed, device="cuda"):
    """Power-law background (exponent beta, mean degree deg) with planted
    G(s, p) blocks; ids permuted at random, orientation random."""
    n, beta = case["n"], case["beta"]
    gen = _generator(seed, device)
    pairs = max(1, int(n * case["deg"] / 2))
    a = 1.0 / (beta - 1.0)
    i0 = _powerlaw_offset(n, a, pairs)
    x = torch.rand(2, pairs, generator=gen, device=device, dtype=torch.float64)
    c0, c1 = i0 ** (1.0 - a), (n + i0) ** (1.0 - a)
    x = ((x * (c1 - c0) + c0) ** (1.0 / (1.0 - a)) - i0).long().clamp_(0, n - 1)
    # the background's heavy vertices and the blocks lie on different ids
    shuffle = torch.randperm(n, generator=gen, device=device)
    us, vs = _blocks(n, case["blocks"], case["s_lo"], case["s_hi"], case["p"], gen)
    u = torch.cat([shuffle[x[0]]] + us)
    v = torch.cat([shuffle[x[1]]] + vs)
    del x
    names = torch.randperm(n, generator=gen, device=device)
    u, v = names[u], names[v]
    flip = torch.rand(len(u), generator=gen, device=device) < 0.5
    return (torch.where(flip, v, u).to(torch.int32).contiguous(), torch.where(flip, u, v).to(torch.int32).contiguous())


def _attachment(case, seed, device="cuda"):
    """Preferential attachment, `mper` edges per new vertex; with probability
    `triad` an edge goes to a random neighbour of the previous edge's target
    instead and closes a triangle."""
    n, mper, triad = case["n"], case["mper"], case["triad"]
    gen = _generator(seed, device)
    v = torch.arange(n, device=device)
    out = torch.empty(mper, n, dtype=torch.int64, device=device)
    for j in range(mper):
        u = torch.rand(n, generator=gen, device=device, dtype=torch.float64)
        t = (u * u * v).long()  # degree of vertex t grows like sqrt(v / t),
        core = torch.randint(0, mper + 1, (n,), generator=gen, device=device)
        t = torch.where(t <= mper, core, t)  # the first vertices alike
        if j > 0 and triad > 0:
            # the target's neighbours: its own earlier edges, and the earlier
            # vertices whose previous edge went to it
            last = out[j - 1]
            key, _ = torch.sort(last * n + v)
            lo = torch.searchsorted(key, last * n)
            cnt = torch.searchsorted(key, last * n + v) - lo
            x = torch.rand(n, generator=gen, device=device, dtype=torch.float64) * (cnt + 1)
            near = key[(lo + x.long()).clamp_(max=n - 1)] % n
            k = torch.randint(0, j, (n,), generator=gen, device=device)
            near = torch.where(x.long() >= cnt, out[k, last], near)
            close = torch.rand(n, generator=gen, device=device) < triad
            t = torch.where(close, near, t)
        out[j] = t.clamp_(max=max(n - 1, 0))
    names = torch.randperm(n, generator=gen, device=device)
    u, w = names[v].repeat(mper), names[out.reshape(-1)]
    return u.to(torch.int32).contiguous(), w.to(torch.int32).contiguous()


def _edges(case, seed, device="cuda"):
    return _powerlaw(case, seed, device) if case["family"] == "powerlaw" else _attachment(case, seed, device)


def _batch_members(case, seed):
    """Uneven small graphs on the host: n spread evenly over its logarithm,
    mean degree 6..20, one to five planted blocks; each an edge-density or a
    triangle-density run with equal chance."""
    rng = np.random.default_rng(int(seed))
    out = []
    for i in range(case["graphs"]):
        n = int(round(case["n_lo"] * (case["n_hi"] / case["n_lo"]) ** ((i + 0.5) / case["graphs"])))
        pairs = max(1, int(n * rng.uniform(6.0, 20.0) / 2))
        a = 1.0 / 1.3
        i0 = _powerlaw_offset(n, a, pairs)
        x = rng.random((2, pairs))
        c0, c1 = i0 ** (1.0 - a), (n + i0) ** (1.0 - a)
        x = np.minimum(((x * (c1 - c0) + c0) ** (1.0 / (1.0 - a)) - i0).astype(np.int64), n - 1)
        us, vs = [x[0]], [x[1]]
        for _ in range(int(rng.integers(1, 6))):
            s = int(rng.integers(4, max(5, min(80, n // 5 + 2))))
            ids = rng.choice(n, size=min(s, n), replace=False)
            hit = np.argwhere(np.triu(rng.random((len(ids), len(ids))) < 0.5, 1))
            us.append(ids[hit[:, 0]])
            vs.append(ids[hit[:, 1]])
        names = rng.permutation(n)
        out.append((n, names[np.concatenate(us)].astype(np.int32), names[np.concatenate(vs)].astype(np.int32),
                    EDGE if rng.random() < 0.5 else TRIANGLE))
    order = rng.permutation(len(out))
    return [out[i] for i in order]


# ------------------------------------------------------------------- cases
def _pl(kind, mode, n, deg, beta, blocks, s_lo, s_hi, p, iters, **kw):
    return dict(kind=kind, mode=mode, family="powerlaw", n=n, deg=float(deg), beta=float(beta), blocks=blocks,
                s_lo=s_lo, s_hi=s_hi, p=float(p), iters=iters, **kw)


def _pa(kind, mode, n, mper, triad, iters, **kw):
    return dict(kind=kind, mode=mode, family="attachment", n=n, mper=mper, triad=float(triad), iters=iters, **kw)


def listed():
    return [
        # the smallest call: one tiny graph from host arrays to its stable
        # groups, where launches, copies and waits are all there is
        dict(_pl("step", EDGE, 61, 8, 2.3, 1, 8, 12, 0.5, 100, host=True), name="tiny_step"),
        # an ordinary small graph (the unit-test workload), kept resident,
        # iterated again with the gap
        dict(_pl("fw", EDGE, 2000, 8, 2.3, 10, 20, 60, 0.5, 200), name="small_fw_edge"),
        # one query of the serving pool's median size, triangle density
        dict(_pl("topk", TRIANGLE, 10_007, 11, 2.3, 5, 20, 80, 0.5, 200, k=5), name="small_topk_tri"),
        # a mid-size graph, edge list to stable groups (the mid-size golden's
        # shape)
        dict(_pl("step", EDGE, 120_000, 20, 2.2, 30, 50, 400, 0.3, 100), name="mid_step_edge"),
        # the same in triangle density on a resident graph
        dict(_pl("groups", TRIANGLE, 100_003, 16, 2.3, 30, 20, 120, 0.5, 200), name="mid_groups_tri"),
        # many small graphs in one launch, half edge half triangle density
        dict(kind="batch", mode=EDGE, family="batch", graphs=768, n_lo=50, n_hi=5000, name="batch_mixed"),
        # a top-k query on a graph beyond one workgroup's size
        dict(_pl("topk", EDGE, 300_000, 14, 2.3, 40, 40, 300, 0.4, 100, k=10), name="mid_topk_edge"),
        # pruning bounds: core numbers of the density sweep's middle graph
        dict(_pa("cores", EDGE, 1_000_000, 8, 0.0, 0), name="large_cores"),
        # triangle listing of the triangle workload's shape
        dict(_pa("listing", TRIANGLE, 1_000_000, 20, 0.6, 0), name="large_listing"),
        # the triangle workload's iterations
        dict(_pa("fw", TRIANGLE, 1_000_000, 20, 0.6, 200), name="large_fw_tri"),
        # the 4-clique workload end to end
        dict(_pl("cliques", CLIQUE4, 1_000_000, 10, 2.2, 200, 20, 200, 0.5, 100), name="large_cliques"),
        # the flagship step: 4M vertices, about 100M edges
        dict(_pl("step", EDGE, 4_000_000, 30, 2.1, 200, 50, 2000, 0.3, 100), name="large_step_edge"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "fw_edge", "fw_tri", "groups", "listing", "cliques", "topk", "batch", "cores"])
    beta = rng.uniform(2.1, 2.5)
    if kind == "step":
        n = _logint(rng, 50, 3_000_000)
        s_hi = max(4, min(2000, n // 5))
        s_lo = max(3, s_hi // 20)
        blocks = max(1, min(150, n // (8 * s_hi)))
        return _pl("step", EDGE, n, rng.uniform(6, 30), beta, blocks, s_lo, s_hi, rng.uniform(0.2, 0.5),
                   rng.randint(50, 100), host=bool(n < 20_000 and rng.random() < 0.5))
    if kind == "fw_edge":
        n = _logint(rng, 300, 2_000_000)
        s_hi = max(4, min(800, n // 6))
        return _pl("fw", EDGE, n, rng.uniform(6, 24), beta, max(1, min(60, n // (8 * s_hi))), max(3, s_hi // 10),
                   s_hi, rng.uniform(0.2, 0.5), rng.randint(50, 200))
    if kind == "fw_tri":
        if rng.random() < 0.5:
            return _pa("fw", TRIANGLE, _logint(rng, 2_000, 900_000), rng.randint(4, 18), rng.uniform(0.2, 0.7),
                       rng.randint(50, 200))
        n = _logint(rng, 300, 500_000)
        return _pl("fw", TRIANGLE, n, rng.uniform(6, 20), beta, max(1, min(40, n // 800)), 10, 100,
                   rng.uniform(0.3, 0.5), rng.randint(50, 200))
    if kind == "groups":
        n = _logint(rng, 200, 400_000)
        mode = rng.choice([EDGE, TRIANGLE])
        return _pl("groups", mode, n, rng.uniform(6, 20), beta, max(1, min(40, n // 1000)), 8, 100,
                   rng.uniform(0.3, 0.5), rng.randint(60, 200))
    if kind == "listing":
        if rng.random() < 0.5:
            return _pa("listing", TRIANGLE, _logint(rng, 1_000, 900_000), rng.randint(4, 20), rng.uniform(0.0, 0.7), 0)
        n = _logint(rng, 200, 1_000_000)
        return _pl("listing", TRIANGLE, n, rng.uniform(6, 20), beta, max(1, min(60, n // 1000)), 8, 150,
                   rng.uniform(0.2, 0.5), 0)
    if kind == "cliques":
        n = _logint(rng, 300, 800_000)
        return _pl("cliques", CLIQUE4, n, rng.uniform(6, 12), beta, max(1, min(120, n // 1000)), 8, 100,
                   rng.uniform(0.3, 0.5), rng.randint(30, 100))
    if kind == "topk":
        n = _logint(rng, 300, 120_000)
        mode = rng.choice([EDGE, TRIANGLE])
        return _pl("topk", mode, n, rng.uniform(6, 14), beta, max(1, min(20, n // 1500)), 10, 100,
                   rng.uniform(0.4, 0.5), 100 if mode == EDGE else 200, k=rng.randint(1, 10))
    if kind == "batch":
        return dict(kind="batch", mode=EDGE, family="batch", graphs=_logint(rng, 24, 600), n_lo=50,
                    n_hi=rng.randint(600, 5000))
    if rng.random() < 0.5:
        return _pa("cores", rng.choice([EDGE, TRIANGLE]), _logint(rng, 1_000, 900_000), rng.randint(2, 12),
                   rng.uniform(0.0, 0.5), 0)
    n = _logint(rng, 300, 500_000)
    return _pl("cores", rng.choice([EDGE, TRIANGLE]), n, rng.uniform(6, 20), beta, max(1, min(30, n // 1000)), 8, 120,
               rng.uniform(0.2, 0.5), 0)


# --------------------------------------------------------------- one pass
def prepare(case, seed):
    L = _library()
    kind, mode = case["kind"], case["mode"]
    st = {"case": case}
    if kind == "batch":
        members = _batch_members(case, seed)
        graphs = [L.lds_create_graph(n, u, v) for n, u, v, _ in members]
        modes = [m[3] for m in members]
        iters = [100 if m == EDGE else 200 for m in modes]
        sizes = [m[0] for m in members]
        st["r"] = torch.zeros(sum(sizes), dtype=torch.float32, device="cuda")
        st["graphs"] = graphs
        st["batch"] = L.lds_batch_create(graphs, modes, iters, r_out=list(torch.split(st["r"], sizes)))
        return st
    u, v = _edges(case, seed)
    n = case["n"]
    if kind in ("step", "listing", "cliques"):
        st["src"], st["dst"] = (u.cpu().numpy(), v.cpu().numpy()) if case.get("host") else (u, v)
    else:
        st["graph"] = L.lds_create_graph(n, u, v)
        if mode != EDGE:
            L.lds_triangles(st["graph"])
    if kind in ("step", "groups", "fw", "cliques"):
        st["r"] = torch.empty(n, dtype=torch.float32, device="cuda")
    return st


def _padded(rows, size, width):
    """Rows of whole numbers as an array of `size` rows (-1 past the last)."""
    a = np.full((size, width), -1, dtype=np.int64)
    if rows:
        a[:len(rows)] = rows[:size]
    return a


def _groups(L, g, case):
    groups, lo, hi = L.lds_stable_groups(g, case["mode"])
    return {"count": len(groups), "groups": _padded(groups, min(case["n"], 16384), 2), "lo": lo, "hi": hi}


def run(state):
    L = _library()
    case = state["case"]
    kind, mode, iters = case["kind"], case["mode"], case.get("iters", 0)
    if kind == "batch":
        L.lds_batch_run(state["batch"])
        return state["r"]
    if kind in ("step", "listing", "cliques"):
        g = L.lds_create_graph(case["n"], state["src"], state["dst"])
        if kind == "listing":
            count, _, per_vertex = L.lds_triangles(g, want_counts=True)
            out = {"triangles": count, "per_vertex": per_vertex}
        else:
            out = {}
            if kind == "cliques":
                out["cliques"] = L.lds_cliques4(g)[0]
            out["r"] = state["r"]
            out["gap"] = L.lds_frank_wolfe(g, mode, iters, r_out=state["r"], want_gap=True)["gap"]
            if kind == "step":
                out.update(_groups(L, g, case))
        g.destroy()
        return out
    g = state["graph"]
    if kind == "cores":
        return L.lds_core_numbers(g, mode)
    if kind == "topk":
        sets = L.lds_topk(g, mode, case["k"], iters)
        member = np.full(case["n"], -1, dtype=np.int32)
        for i, (ids, _) in enumerate(sets):
            member[ids] = i
        return {"member": member,
                "sets": _padded([(len(ids), d.numerator, d.denominator) for ids, d in sets], case["k"], 3)}
    out = {"r": state["r"],
           "gap": L.lds_frank_wolfe(g, mode, iters, r_out=state["r"], want_gap=True)["gap"]}
    if kind == "groups":
        out.update(_groups(L, g, case))
    return out


# ------------------------------------------------------------------- sizes
def _expected(case):
    """Expected numbers of edges, triangles and 4-cliques of a case's graph
    (the planted blocks' in the mean; the background's triangles and cliques,
    which hang on its largest degrees, are left out: a lower bound)."""
    if case["family"] == "attachment":
        return case["n"] * case["mper"], case["n"] * case["mper"] * case["triad"], 0.0
    s = (case["s_lo"] + case["s_hi"]) / 2.0
    spread = (case["s_hi"] - case["s_lo"]) ** 2 / 12.0
    s2, s3 = s * s + spread, s ** 3 + 3 * s * spread
    s4 = s ** 4 + 6 * s * s * spread + (case["s_hi"] - case["s_lo"]) ** 4 / 80.0
    p, b = case["p"], case["blocks"]
    return case["n"] * case["deg"] / 2.0 + b * p * s2 / 2.0, b * p ** 3 * s3 / 6.0, b * p ** 6 * s4 / 24.0


def work(case):
    if case["kind"] == "batch":
        mean_n = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        m = case["graphs"] * mean_n * 8.0
        return {"bytes": 8.0 * m + 4.0 * case["graphs"] * mean_n, "flops": 4.0 * m * 150}
    n, kind = case["n"], case["kind"]
    m, t, q = _expected(case)
    patterns = {EDGE: m, TRIANGLE: t, CLIQUE4: q}[case["mode"]]
    out_bytes = {"step": 20.0 * n, "groups": 20.0 * n, "fw": 4.0 * n, "listing": 8.0 * n, "cliques": 4.0 * n,
                 "topk": 8.0, "cores": 8.0 * n}[kind]
    # per pattern member and iteration one compare and one addition; listing
    # and peeling touch every edge (pattern) member once
    return {"bytes": 8.0 * m + out_bytes, "flops": 2.0 * case["mode"] * max(patterns, 1.0) * max(case["iters"], 1)}


# ------------------------------------------------------------- exact values
def _simple(n, u, v):
    """Canonical edges (u < v) of a pair list, without loops or duplicates."""
    u, v = u.long(), v.long()
    key = torch.unique((torch.minimum(u, v) * n + torch.maximum(u, v))[u != v])
    return torch.div(key, n, rounding_mode="floor"), key % n


def _triangles(n, u, v, limit):
    """Triangles as three vertex arrays, by wedges from the endpoint of
    smaller degree; None past `limit` wedges."""
    deg = torch.bincount(u, minlength=n) + torch.bincount(v, minlength=n)
    swap = (deg[v] < deg[u]) | ((deg[v] == deg[u]) & (v < u))
    a, b = torch.where(swap, v, u), torch.where(swap, u, v)
    key, _ = torch.sort(a * n + b)
    a, b = torch.div(key, n, rounding_mode="floor"), key % n
    cnt = torch.bincount(a, minlength=n)
    start = torch.cumsum(cnt, 0) - cnt
    pos = torch.arange(len(a), device=a.device) - start[a]
    later = cnt[a] - pos - 1  # pairs (this edge, a later edge of the same vertex)
    total = int(later.sum())
    if total > limit:
        return None
    first = torch.repeat_interleave(torch.arange(len(a), device=a.device), later)
    off = torch.arange(total, device=a.device) - (torch.cumsum(later, 0) - later)[first]
    second = first + 1 + off
    x, y = b[first], b[second]
    swap = (deg[y] < deg[x]) | ((deg[y] == deg[x]) & (y < x))
    want = torch.where(swap, y * n + x, x * n + y)
    at = torch.searchsorted(key, want).clamp_(max=max(len(key) - 1, 0))
    hit = key[at] == want
    return a[first][hit], x[hit], y[hit]


def _exact_fw(n, members, mode, iters):
    """Loads after `iters` iterations and the gap of every iteration, from
    64-bit integer numerators over the common denominator."""
    c = {EDGE: 1, TRIANGLE: 3}[mode]
    dev = members[0].device
    A = torch.zeros(n, dtype=torch.int64, device=dev)
    for m in members:
        A += torch.bincount(m, minlength=n) * (1 if mode == EDGE else 2)
    gaps = []
    for i in range(1, iters + 1):
        D = c * i * (i + 1)
        # the member of smallest load, ties to the larger id
        best, load = members[0], A[members[0]]
        for m in members[1:]:
            lm = A[m]
            take = (lm < load) | ((lm == load) & (m > best))
            best, load = torch.where(take, m, best), torch.where(take, lm, load)
        r = A.double() / D
        gaps.append(2.0 * ((r * r).sum() - (load.double() / D).sum()))
        A = A + (c * (i + 1) * (i + 2) - D) * torch.bincount(best, minlength=n)
    gap = torch.stack(gaps).cpu().numpy() if gaps else np.empty(0)
    return A.double() / (c * (iters + 1) * (iters + 2)), gap


def exact(case, seed):
    kind, mode = case["kind"], case["mode"]
    if kind not in ("step", "groups", "fw") or mode == CLIQUE4:
        return None
    n = case["n"]
    u, v = _simple(n, *_edges(case, seed))
    members = (u, v) if mode == EDGE else _triangles(n, u, v, 400_000_000)
    if members is None or len(members[0]) * case["iters"] > 10 ** 11 or len(members[0]) == 0:
        return None
    r, gap = _exact_fw(n, members, mode, case["iters"])
    out = {"r": r, "gap": gap}
    if kind != "fw":
        out.update({"count": None, "groups": None, "lo": None, "hi": None})  # whole numbers: equal, not near
    return out
