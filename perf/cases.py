"""The work that programs give this library, as cases that can be timed.

A case names one use of a public entry point with its sizes; `prepare` makes
what the program holds before the call (graph handle, workspace, plan, server),
`run` is one pass, `work` what the pass cannot do without and `exact` the
results from plain torch.  Graphs are R-MAT ((a, b, c, d) = (.57, .19, .19,
.05), repeats removed, vertices relabelled) or Erdős–Rényi without self-loops,
given as the int32 CSR of in-edges, the recipes of the package's workloads;
c = 0.6 and delta = 1e-3 throughout, as there.
"""
import math

import numpy as np
import torch

from paper_2304_04015_amd import simrank as S

C, DELTA, CAP = 0.6, 1e-3, 64
ABCD = (0.57, 0.19, 0.19, 0.05)
MASK = 0xFFFFFFFF


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # The smallest call: the tiny workload (n = 500, R = 2000, 32 steps),
        # synchronous, host arrays back; what a notebook or a test does.
        {"name": "tiny_call", "kind": "call", "graph": "er", "n": 500, "deg": 5, "eps": 0.05,
         "R": 2000, "cap": 32},
        # A small graph from the low end of the batching mix, odd size, queried
        # again and again through one workspace with device outputs.
        {"name": "small_async", "kind": "async", "graph": "rmat", "n": 5003, "deg": 11, "eps": 0.05},
        # An ordinary synchronous query of the paper's statement (G, s, c, eps,
        # delta) -> estimates, on a graph of some tens of thousands of nodes.
        {"name": "small_call", "kind": "call", "graph": "rmat", "n": 40000, "deg": 16, "eps": 0.05},
        # The headline query: n = 2^20, average degree 16, eps = 0.02.
        {"name": "medium", "kind": "async", "graph": "rmat", "n": 1 << 20, "deg": 16, "eps": 0.02},
        # The serving graph (n = 2^22), the lone plain query it is compared with.
        {"name": "large", "kind": "async", "graph": "rmat", "n": 1 << 22, "deg": 16, "eps": 0.02},
        # Stitched walks from a resident segment index (2^4 steps a segment).
        {"name": "stitched", "kind": "stitched", "graph": "rmat", "n": 1 << 20, "deg": 16,
         "eps": 0.02, "seg_log2": 4},
        # Algorithms 1-2's length-stratified estimator with its own z and cap.
        {"name": "stratified", "kind": "stratified", "graph": "rmat", "n": 1 << 18, "deg": 16,
         "eps": 0.02},
        # 32 sources with one walk seed: a kept plan, run and read back.
        {"name": "group", "kind": "group", "graph": "rmat", "n": 1 << 18, "deg": 16, "eps": 0.02,
         "members": 32},
        # A batch call over graphs of mixed sizes, a seed per query, eps drawn
        # from the three accuracy levels of the batching mix.
        {"name": "batch_mix", "kind": "batch", "n_min": 1 << 12, "n_max": 150000, "graphs": 4,
         "queries": 16, "deg": 16, "eps_min": 0.01},
        # Meet detection by sorted tuples for several sources at once.
        {"name": "tuples", "kind": "tuples", "graph": "rmat", "n": 16384, "deg": 16, "eps": 0.05,
         "members": 8},
        # A program's start: load the CSR, build the stitched index, first
        # stitched query, free.
        {"name": "cold_start", "kind": "cold", "graph": "rmat", "n": 300007, "deg": 16, "eps": 0.05,
         "seg_log2": 3},
        # A burst of requests at a server (continuous batching), eps mixed.
        {"name": "serve", "kind": "serve", "graph": "rmat", "n": 1 << 18, "deg": 16, "eps": 0.02,
         "requests": 12},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["call", "async", "async", "stitched", "stratified", "group", "batch",
                       "tuples", "cold", "serve"])
    eps = rng.choice([0.05, 0.02, 0.01])
    deg = rng.randint(8, 32)
    if kind == "call":
        if rng.random() < 0.3:
            return {"kind": kind, "graph": "er", "n": _log_uniform(rng, 100, 5000),
                    "deg": rng.randint(3, 8), "eps": 0.05, "R": rng.randint(500, 4000), "cap": 32}
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1000, 200000), "deg": deg,
                "eps": rng.choice([0.05, 0.02])}
    if kind == "async":
        # walks per node grow 25-fold from eps = 0.05 to 0.01
        hi = {0.05: 1 << 22, 0.02: 1 << 21, 0.01: 1 << 19}[eps]
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1 << 12, hi), "deg": deg, "eps": eps}
    if kind == "stitched":
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1 << 12, 1 << 20),
                "deg": rng.randint(8, 16), "eps": rng.choice([0.05, 0.02]), "seg_log2": rng.choice([3, 4])}
    if kind == "stratified":
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1 << 12, 1 << 19), "deg": deg,
                "eps": rng.choice([0.05, 0.02])}
    if kind == "group":
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1 << 12, 1 << 18), "deg": deg,
                "eps": rng.choice([0.05, 0.02]), "members": rng.randint(2, 32)}
    if kind == "batch":
        return {"kind": kind, "n_min": 1 << 12, "n_max": _log_uniform(rng, 1 << 13, 150000),
                "graphs": rng.randint(2, 6), "queries": rng.randint(4, 24), "deg": deg, "eps_min": 0.01}
    if kind == "tuples":
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1000, 50000), "deg": deg,
                "eps": 0.05, "members": rng.randint(1, 16)}
    if kind == "cold":
        return {"kind": kind, "graph": "rmat", "n": _log_uniform(rng, 1 << 12, 300007),
                "deg": rng.randint(8, 16), "eps": 0.05, "seg_log2": rng.choice([2, 3, 4])}
    return {"kind": "serve", "graph": "rmat", "n": _log_uniform(rng, 1 << 12, 1 << 18), "deg": deg,
            "eps": 0.02, "requests": rng.randint(2, 12)}


# -------------------------------------------------------------------- the inputs

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _rng(seed, salt):
    return np.random.Generator(np.random.PCG64([int(seed), int(salt)]))


def _edges(graph, n, deg, gen, dev):
    if graph == "er":
        k = torch.poisson(torch.full((n,), float(deg), device=dev), generator=gen).long()
        dst = torch.repeat_interleave(torch.arange(n, device=dev), k)
        src = torch.randint(0, n, (dst.numel(),), generator=gen, device=dev)
        keep = src != dst
        return src[keep], dst[keep]
    scale = max(1, (n - 1).bit_length())
    want, have, us, vs = n * deg, 0, [], []
    a, ab, abc = ABCD[0], ABCD[0] + ABCD[1], ABCD[0] + ABCD[1] + ABCD[2]
    while have < want:
        e = max(want - have, 4096)
        u = torch.zeros(e, dtype=torch.int64, device=dev)
        v = torch.zeros(e, dtype=torch.int64, device=dev)
        for bit in range(scale):
            r = torch.rand(e, generator=gen, device=dev)
            u |= (r >= ab).long() << bit
            v |= (((r >= a) & (r < ab)) | (r >= abc)).long() << bit
        keep = (u < n) & (v < n)
        us.append(u[keep])
        vs.append(v[keep])
        have += us[-1].numel()
    u, v = torch.cat(us)[:want], torch.cat(vs)[:want]
    perm = torch.randperm(n, generator=gen, device=dev)
    return perm[u], perm[v]


def _csr(graph, n, deg, seed):
    """In-edge CSR (row v lists the in-neighbours of v, ascending), host int32."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1000003 + n * 31 + deg)
    src, dst = _edges(graph, n, deg, gen, dev)
    key = torch.unique(dst * n + src)
    counts = torch.bincount(torch.div(key, n, rounding_mode="floor"), minlength=n)
    off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    off[1:] = torch.cumsum(counts, 0)
    return off.to(torch.int32).cpu().numpy(), (key % n).to(torch.int32).cpu().numpy()


def _sources(off, count, seed):
    """Sources drawn with probability proportional to in-degree, as requests arrive."""
    d = np.diff(off.astype(np.int64)).astype(np.float64)
    return [int(x) for x in _rng(seed, 7).choice(d.size, size=count, p=d / d.sum())]


def _batch_specs(case):
    """Graph sizes spread over the logarithm of the range, and each query's (graph, eps)."""
    steps, span = case["graphs"] - 1, case["n_max"] / case["n_min"]
    ns = [int(case["n_min"] * span ** (i / steps)) | 1 for i in range(steps + 1)]
    eps = [e for e in (0.05, 0.02, 0.01) if e >= case["eps_min"]]
    # the accuracy levels in turn, the graphs from the largest down
    return ns, [(i % len(ns), eps[i % len(eps)]) for i in range(case["queries"])]


def _plain_query(case, s, seed):
    return S.make_query(s, c=C, eps=case["eps"], delta=DELTA, seed=seed,
                        walk_cap=case.get("cap", CAP), R=case.get("R", 0))


def prepare(case, seed):
    kind = case["kind"]
    wseed = 0x2304040150000000 + int(seed)
    if kind == "batch":
        ns, mix = _batch_specs(case)
        csrs = [_csr("rmat", n, case["deg"], seed * 16 + i) for i, n in enumerate(ns)]
        graphs = [S.simrank_load_graph(n, off, src) for n, (off, src) in zip(ns, csrs)]
        qs = [S.make_query(_sources(csrs[g][0], 1, seed * 64 + i)[0], c=C, eps=e, delta=DELTA,
                           seed=wseed + 1000 * i, graph=g) for i, (g, e) in enumerate(mix)]
        return {"kind": kind, "graphs": graphs, "queries": qs}
    n = case["n"]
    off, src = _csr(case["graph"], n, case["deg"], seed)
    st = {"kind": kind, "n": n, "case": case, "wseed": wseed}
    if kind == "cold":
        st.update(off=off, src=src, s=_sources(off, 1, seed)[0])
        return st
    g = st["g"] = S.simrank_load_graph(n, off, src)
    count = case.get("members") or case.get("requests") or 1
    sources = _sources(off, count, seed)
    if kind == "call":
        st["q"] = _plain_query(case, sources[0], wseed)
    elif kind in ("async", "stitched"):
        q = _plain_query(case, sources[0], wseed)
        if kind == "stitched":
            S.simrank_build_index(g, seg_log2=case["seg_log2"], kappa=1.0, c=C, seed=wseed + 1)
            q.mode = S.MODE_STITCHED
        p = S.simrank_derive_params(q, n)
        st["q"], st["ws"] = q, S.simrank_workspace_create(g, p.R, p.L)
        st["out"] = torch.zeros(n, dtype=torch.float64, device="cuda")
        st["cnt"] = torch.zeros(n, dtype=torch.int32, device="cuda")
    elif kind == "stratified":
        q = S.make_stratified_query(sources[0], c=C, eps=case["eps"], seed=wseed, delta=DELTA)
        p = S.simrank_derive_stratified(q, n)
        st["q"], st["ws"] = q, S.simrank_workspace_create(g, p.N, p.phi)
        st["out"] = torch.zeros(n, dtype=torch.float64, device="cuda")
        st["out_n"] = torch.zeros(n, dtype=torch.float64, device="cuda")
        st["wsum"] = torch.zeros(n, dtype=torch.int64, device="cuda")
    elif kind == "group":
        st["plan"] = S.BatchPlan([g], [_plain_query(case, s, wseed) for s in sources])
    elif kind == "tuples":
        st["queries"] = [_plain_query(case, s, wseed) for s in sources]
    elif kind == "serve":
        levels = (case["eps"], 0.05)
        st["queries"] = [S.make_query(s, c=C, eps=levels[i % 2], delta=DELTA, seed=wseed + 1000 * i)
                         for i, s in enumerate(sources)]
        p = S.simrank_derive_params(st["queries"][0], n)
        st["server"] = S.Server(g, max_slots=16, max_R=p.R, max_L=p.L, hbm_budget=1 << 30)
    return st


# ---------------------------------------------------------------------- one pass

def run(st):
    kind = st["kind"]
    if kind == "batch":
        outs, cnts, _ = S.simrank_batch(st["graphs"], st["queries"])
        return {"out": outs, "counts": cnts}
    if kind == "call":
        out, cnt, _ = S.simrank_single_source_ex(st["g"], st["q"])
        return {"out": out, "counts": cnt}
    if kind in ("async", "stitched"):
        S.simrank_single_source_async(st["g"], st["q"], st["ws"], st["out"], st["cnt"],
                                      torch.cuda.current_stream())
        return {"out": st["out"], "counts": st["cnt"]}
    if kind == "stratified":
        S.simrank_stratified_async(st["g"], st["q"], st["ws"], st["out"], st["out_n"], st["wsum"],
                                   torch.cuda.current_stream())
        return {"out": st["out"], "out_n": st["out_n"], "wsum": st["wsum"]}
    if kind == "group":
        plan = st["plan"]
        plan.run(torch.cuda.current_stream())
        plan.wait()
        return {"out": [plan.read(i, want_counts=False)[0] for i in range(len(plan.queries))]}
    if kind == "tuples":
        sums, _ = S.simrank_tuple_meets(st["g"], st["queries"])
        return {"sums": sums}
    if kind == "cold":
        case = st["case"]
        g = S.simrank_load_graph(st["n"], st["off"], st["src"])
        S.simrank_build_index(g, seg_log2=case["seg_log2"], kappa=1.0, c=C, seed=st["wseed"] + 1)
        q = _plain_query(case, st["s"], st["wseed"])
        q.mode = S.MODE_STITCHED
        out, cnt, _ = S.simrank_single_source_ex(g, q)
        g.free()
        return {"out": out, "counts": cnt}
    tickets = [st["server"].submit(q) for q in st["queries"]]
    res = [st["server"].wait(t) for t in tickets]
    return {"out": [r[0] for r in res], "counts": [r[1] for r in res]}


# ------------------------------------------------------------- what it comes to

def _walks(case, eps=None):
    """Walks per node: the Hoeffding count; Algorithm 2's z for stratified queries."""
    eps = case["eps"] if eps is None else eps
    if case["kind"] == "stratified":
        return math.log(2.0 * case["n"]) / (2.0 * (eps - 3.0 / case["n"]) ** 2)
    return case.get("R") or math.ceil(math.log(2 / DELTA) / (2 * (eps - C ** (CAP + 1)) ** 2))


def work(case):
    """The graph (8 bytes an edge: neighbour and degree) read and the results
    written once; the integer operations of the draws (ten Philox rounds of two
    products and four more operations, and the pick) of the steps a pair (v, j)
    needs: c / (1 - c) on average until one of its two walks has ended, or the
    walk's own length sqrt(c) / (1 - sqrt(c)) where many sources share it.
    About half of an R-MAT graph's nodes have in-edges."""
    ops_per_step = 10 * 6 + 4
    lone, full = C / (1 - C), math.sqrt(C) / (1 - math.sqrt(C))
    if case["kind"] == "batch":
        ns, mix = _batch_specs(case)
        steps = sum(0.5 * ns[g] * _walks(case, e) * lone for g, e in mix)
        return {"bytes": sum(8 * n * case["deg"] for n in ns) + sum(12 * ns[g] for g, _ in mix),
                "flops": int(ops_per_step * steps)}
    n = case["n"]
    active = n * (1.0 if case["graph"] == "er" else 0.5)
    members = case.get("members", 1)
    out = {"stratified": 24 * n, "tuples": 8 * n * members, "group": 8 * n * members}.get(case["kind"], 12 * n)
    steps = active * _walks(case) * (full if members > 1 else lone)
    if case["kind"] == "serve":
        steps = sum(active * _walks(case, e) * lone for e in [(case["eps"], 0.05)[i % 2] for i in range(case["requests"])])
        out = 12 * n * case["requests"]
    bytes_ = 8 * n * case["deg"] + out
    if case["kind"] == "cold":
        # the CSR arrives from the host; one segment and its chain per edge
        per_slot = 4 * (1 << case["seg_log2"]) + 4 * (64 >> case["seg_log2"]) + 5
        bytes_ += n * case["deg"] * (4 + per_slot)
        steps += n * case["deg"] * full
    return {"bytes": bytes_, "flops": int(ops_per_step * steps)}


def _philox(c0, c1, c2, key):
    """Words 0 and 1 of Philox4x32-10 on counters (c0, c1, c2, 0), int64 tensors."""
    k0, k1 = key & MASK, key >> 32
    c3 = torch.zeros_like(c0)
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((p1 >> 32) & MASK) ^ c1 ^ k0, p1 & MASK, ((p0 >> 32) & MASK) ^ c3 ^ k1, p0 & MASK)
        k0, k1 = (k0 + 0x9E3779B9) & MASK, (k1 + 0xBB67AE85) & MASK
    return c0, c1


def _plain_estimate(n, off, src, s, R, cap, key):
    """s_hat(s, .) of plain sqrt(c)-walks, walked pair by pair in torch."""
    dev = _device()
    off, src = torch.from_numpy(off).to(dev).long(), torch.from_numpy(src).to(dev).long()
    deg = off[1:] - off[:-1]
    T = min(math.floor(math.sqrt(C) * 2.0 ** 32), 2 ** 32 - 1)

    def step(node, v, j, t):
        x0, x1 = _philox(v, j, torch.full_like(v, t), key)
        go = (x0 < T) & (deg[node] > 0)
        at = off[node] + ((x1 * deg[node]) >> 32)
        return go, src[torch.where(go, at, torch.zeros_like(at))]

    j0 = torch.arange(R, device=dev)
    path, alive, node = [], torch.ones(R, dtype=torch.bool, device=dev), torch.full((R,), s, device=dev)
    for t in range(1, cap + 1):
        go, nxt = step(node, torch.full_like(j0, s), j0, t)
        alive = alive & go
        node = torch.where(alive, nxt, node)
        path.append(torch.where(alive, nxt, torch.full_like(nxt, -1)))
        if not bool(alive.any()):
            break
    counts = torch.zeros(n, dtype=torch.int64, device=dev)
    vs = torch.nonzero(deg > 0).flatten()
    block = max(1, (1 << 23) // R)
    for b in range(0, vs.numel(), block):
        v = vs[b:b + block].repeat_interleave(R)
        j = j0.repeat(vs[b:b + block].numel())
        cur = v
        for t, there in enumerate(path, 1):
            live = there[j] >= 0
            v, j, cur = v[live], j[live], cur[live]
            if v.numel() == 0:
                break
            go, nxt = step(cur, v, j, t)
            v, j, cur = v[go], j[go], nxt[go]
            met = cur == there[j]
            counts += torch.bincount(v[met], minlength=n)
            v, j, cur = v[~met], j[~met], cur[~met]
    est = counts.double() / R
    est[s] = 1.0
    return est.cpu()


def exact(case, seed):
    """Plain queries small enough to be walked in torch; no value elsewhere."""
    if case["kind"] not in ("call", "async") or case["n"] * _walks(case) > 1 << 26:
        return None
    off, src = _csr(case["graph"], case["n"], case["deg"], seed)
    s = _sources(off, 1, seed)[0]
    est = _plain_estimate(case["n"], off, src, s, int(_walks(case)), case.get("cap", CAP),
                          0x2304040150000000 + int(seed))
    return {"out": est, "counts": None}
