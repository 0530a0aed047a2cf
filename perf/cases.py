"""The work a user of this library has it do, as measurable cases.

A case is a dict of plain values; prepare() makes what a program holds before
the call (a context, the resident graph, registered queries, batches), run()
is one pass through the public calls, work() the bytes a pass cannot do
without.  Graphs are seeded R-MAT (a=.57, b=.19, c=.19, d=.05, the skew of the
social graphs the paper evaluates) or Erdos-Renyi edge lists.

Everything here is an exact integer: counts, per-stage counters, sorted rows,
index arrays.
"""
import math

import numpy as np
import torch

import paper_1802_03760_amd as gj

QUERIES = {
    "triangle": (3, [(0, 1), (1, 2), (0, 2)]),
    "cyclic_triangle": (3, [(0, 1), (1, 2), (2, 0)]),
    "clique4": (4, [(0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3)]),
    "diamond": (4, [(0, 1), (0, 2), (1, 3), (2, 3)]),
    "cycle4": (4, [(0, 1), (1, 2), (2, 3), (3, 0)]),
    "house": (5, [(0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3), (1, 4), (2, 4)]),
    "clique5": (5, [(i, j) for i in range(5) for j in range(i + 1, 5)]),
}
LESS = {"triangle": [(0, 1), (1, 2)], "clique4": [(0, 1), (1, 2), (2, 3)]}
BATCH_MIX = ["clique4", "diamond", "clique4", "diamond", "triangle", "cycle4"]
# One side stream for every state, as one program has it: the caching
# allocator can then hand a released block to the next context.
_stream = []


def listed():
    return [
        # The smallest graph in use: a count on 20,000 edges, where launches,
        # host reads and start-up work are all there is.
        {"name": "er2000_triangle", "kind": "count", "query": "triangle", "graph": "er", "vertices": 2000,
         "draws": 20000},
        # A query without a kernel of its own (five attributes, the generic
        # stages) on a small graph of odd size.
        {"name": "rmat4099_house", "kind": "count", "query": "house", "graph": "rmat", "vertices": 4099,
         "draws": 65537},
        # The evaluation's triangle count at the size of its LiveJournal runs.
        {"name": "rmat22_triangle", "kind": "count", "query": "triangle", "graph": "rmat", "vertices": 1 << 22,
         "draws": 1 << 26},
        # Every triangle listed, sorted, into device memory.
        {"name": "rmat20_triangle_rows", "kind": "rows", "query": "triangle", "graph": "rmat", "vertices": 1 << 20,
         "draws": 1 << 24},
        # Whole counts of the four-attribute shapes of the evaluation.
        {"name": "rmat18_diamond", "kind": "count", "query": "diamond", "graph": "rmat", "vertices": 1 << 18,
         "draws": 1 << 22},
        {"name": "rmat600011_cycle4", "kind": "count", "query": "cycle4", "graph": "rmat", "vertices": 600011,
         "draws": 9000001},
        # Cliques of an undirected graph, each once: degree-ordered builds.
        {"name": "rmat20_clique4_oriented", "kind": "count", "query": "clique4", "graph": "rmat",
         "vertices": 1 << 20, "draws": 1 << 24, "degree_order": True},
        {"name": "rmat300007_clique5_oriented", "kind": "count", "query": "clique5", "graph": "rmat",
         "vertices": 300007, "draws": 4500001, "degree_order": True},
        # Many short requests of mixed queries served as one batch.
        {"name": "rmat22_batch256", "kind": "batch", "graph": "rmat", "vertices": 1 << 22, "draws": 1 << 26,
         "requests": 256, "width": 100},
        # Triangle maintenance: a small batch arrives, and its inverse as it
        # expires from a sliding window.
        {"name": "rmat22_update1000", "kind": "update", "query": "triangle", "graph": "rmat", "vertices": 1 << 22,
         "draws": 1 << 26, "size": 1000},
        # The same with a large batch, the changed triangles listed.
        {"name": "rmat20_update30011_rows", "kind": "update", "query": "triangle", "graph": "rmat",
         "vertices": 1 << 20, "draws": 1 << 24, "size": 30011, "rows": True},
        # The index build a new graph begins with, from device arrays.
        {"name": "rmat22_build", "kind": "build", "graph": "rmat", "vertices": 1 << 22, "draws": 60000000},
    ]


def draw(rng):
    def size(lo, hi):  # vertices 2^lo .. 2^hi, any number; 8 to 16 draws each
        n = int(2.0 ** rng.uniform(lo, hi))
        return {"graph": "rmat", "vertices": n, "draws": int(n * rng.uniform(8, 16))}

    kind = rng.choice(["tri", "tri", "er", "generic", "rows", "twopath", "twopath", "clique4", "clique4", "clique5",
                       "batch", "update", "update", "build"])
    if kind == "tri":
        c = {"kind": "count", "query": rng.choice(["triangle", "triangle", "cyclic_triangle"]), **size(11, 22)}
        if rng.random() < 0.3:
            c["degree_order"] = True
        return c
    if kind == "er":
        n = int(2.0 ** rng.uniform(7, 16))
        return {"kind": "count", "query": rng.choice(["triangle", "cyclic_triangle", "clique4", "diamond", "cycle4"]),
                "graph": "er", "vertices": n, "draws": int(n * rng.uniform(4, 16))}
    if kind == "generic":
        c = {"kind": "count", "query": "house", **size(9, 13)}
        if rng.random() < 0.4:
            c["factorise"] = True
        return c
    if kind == "rows":
        q = rng.choice(["triangle", "triangle", "cyclic_triangle", "clique4", "diamond"])
        c = {"kind": "rows", "query": q, **(size(10, 20) if "triangle" in q else size(9, 11.5))}
        if c["vertices"] <= 1 << 14 and "triangle" in q and rng.random() < 0.5:
            c["host"] = True
        return c
    if kind == "twopath":
        return {"kind": "count", "query": rng.choice(["diamond", "cycle4"]), **size(11, 19)}
    if kind == "clique4":
        form = rng.choice(["oriented", "oriented", "directed", "less"])
        c = {"kind": "count", "query": "clique4", **(size(12, 20) if form == "oriented" else size(11, 17))}
        if form == "oriented":
            c["degree_order"] = True
        if form == "less":
            c.update(undirected=True, less=True)
        return c
    if kind == "clique5":
        return {"kind": "count", "query": "clique5", "degree_order": True, **size(12, 18.5)}
    if kind == "batch":
        return {"kind": "batch", "requests": int(2.0 ** rng.uniform(3, 8)), "width": int(2.0 ** rng.uniform(2, 7)),
                **size(16, 22)}
    if kind == "update":
        c = {"kind": "update", "query": rng.choice(["triangle", "triangle", "cyclic_triangle"]),
             "size": int(10.0 ** rng.uniform(1, 5)), **size(16, 22)}
        r = rng.random()
        if r < 0.3 and c["size"] <= 32000:
            c["rows"] = True
        if r > 0.7:
            c["lsm"] = True
        return c
    c = {"kind": "build", **size(12, 22)}
    c["draws"] = int(c["draws"] * 0.8)
    r = rng.random()
    if r < 0.25:
        c["degree_order"] = True
    elif r < 0.5:
        c["undirected"] = True
    return c


# ------------------------------------------------------------------- inputs


def _rmat(n, m, gen):
    """At most m R-MAT draws over n vertices (those beyond n dropped), repeats
    and self-loops kept, as two int32 device tensors."""
    src = torch.zeros(m, dtype=torch.int32, device="cuda")
    dst = torch.zeros(m, dtype=torch.int32, device="cuda")
    for _ in range(max(1, (n - 1).bit_length())):
        u = torch.rand(m, device="cuda", generator=gen)
        src.mul_(2).add_(u >= 0.76)
        dst.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    keep = (src < n) & (dst < n)
    return src[keep].contiguous(), dst[keep].contiguous()


def _distinct_pairs(n, m, gen):
    """m distinct pairs from R-MAT draws, a sixteenth of them both ways and a
    sixteenth twice, in any order: an edge list whose indexes have the same
    sizes whatever the seed."""
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < m:
        s, d = _rmat(n, 2 * m, gen)
        lo, hi = torch.minimum(s, d), torch.maximum(s, d)
        keys = torch.unique(torch.cat([keys, _keys(lo, hi, n)[lo != hi]]))
    keys = keys[torch.randperm(keys.numel(), device="cuda", generator=gen)[:m]]
    s, d = (keys // n).to(torch.int32), (keys % n).to(torch.int32)
    flip = torch.rand(m, device="cuda", generator=gen) < 0.5
    s, d = torch.where(flip, d, s), torch.where(flip, s, d)
    k = m // 16
    s, d = torch.cat([s, d[:k], s[m - k:]]), torch.cat([d, s[:k], d[m - k:]])
    mix = torch.randperm(s.numel(), device="cuda", generator=gen)
    return s[mix].contiguous(), d[mix].contiguous()


def _edges(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, m = case["vertices"], case["draws"]
    if case["graph"] == "er":
        return tuple(torch.randint(0, n, (m,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(2))
    if case["kind"] == "build":
        return _distinct_pairs(n, m, gen)
    return _rmat(n, m, gen)


def _keys(src, dst, n):
    return src.to(torch.int64) * n + dst.to(torch.int64)


def _edge_set(src, dst, n):
    k = torch.unique(_keys(src, dst, n))
    return k[k // n != k % n]


def _member(sorted_keys, k):
    at = torch.searchsorted(sorted_keys, k).clamp_(max=sorted_keys.numel() - 1)
    return sorted_keys[at] == k


def _update_batches(case, seed, src, dst):
    """A batch of fresh draws with a tenth deletions of present edges (some
    insertions are of edges already there, as in a real stream), and the batch
    that takes its effect back."""
    n, b = case["vertices"], case["size"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1000003)
    base = _edge_set(src, dst, n)
    nd = max(1, b // 10)
    pick = torch.randint(0, base.numel(), (nd,), device="cuda", generator=gen)
    dels = torch.unique(base[pick])
    s, d = _rmat(n, max(8, 2 * b), gen)
    ins = _keys(s[:b - nd], d[:b - nd], n)
    ins = ins[~torch.isin(ins, dels)]
    real = torch.unique(ins[ins // n != ins % n])
    real = real[~_member(base, real)]

    def rows(up, down):
        k = torch.cat([up, down])
        sign = torch.cat([torch.ones_like(up), -torch.ones_like(down)])
        mix = torch.randperm(k.numel(), device="cuda", generator=gen)
        k, sign = k[mix], sign[mix]
        return ((k // n).cpu().numpy().astype(np.uint32), (k % n).cpu().numpy().astype(np.uint32),
                sign.cpu().numpy().astype(np.int8))

    return rows(ins, dels), rows(dels, real)


def _rows_room(case):
    """Rows a result buffer holds: what an R-MAT graph of this size gives, with
    room; the same for every seed."""
    s, ef = math.log2(case["vertices"]), case["draws"] / case["vertices"] / 16.0
    if case["kind"] == "update":  # three triangles per edge and triangle of the graph
        return int(3 * case["size"] * 106 * 1.1 ** (s - 20) * ef) + 4096
    per = {"triangle": (5.7e8, 2.207, 20, 2), "cyclic_triangle": (5.7e8, 2.207, 20, 2),
           "clique4": (1.2e8, 2.72, 14, 3), "diamond": (8.3e8, 2.95, 14, 3)}[case["query"]]
    return int(2 * per[0] * per[1] ** (s - per[2]) * ef ** per[3]) + 4096


def prepare(case, seed):
    if not _stream:
        _stream.append(torch.cuda.Stream())
    src, dst = _edges(case, seed)
    torch.cuda.synchronize()
    ctx = gj.Context(0, _stream[0], allocator="torch")
    st = {"case": case, "ctx": ctx}
    flags = {"undirected": case.get("undirected", False), "degree_order": case.get("degree_order", False)}
    if case["kind"] == "build":
        st.update(src=src, dst=dst, flags=flags, graph=None)
        return st
    if case.get("factorise"):
        ctx.set_option("factorise", 1)
    if case.get("lsm"):
        ctx.set_option("lsm_updates", 1)
    st["graph"] = g = gj.Graph(ctx, src, dst, case["vertices"], **flags)
    if case["kind"] == "batch":
        rng = np.random.default_rng(seed)
        qs = {k: gj.Query(ctx, *QUERIES[k]) for k in BATCH_MIX}
        edges = g.info(degrees=False)["edges"]
        reqs = []
        for i in range(case["requests"]):
            lo = int(rng.integers(0, edges))
            reqs.append((qs[BATCH_MIX[i % len(BATCH_MIX)]], lo,
                         min(edges, lo + int(np.exp(rng.uniform(0, np.log(case["width"])))))))
        st["requests"] = reqs
        return st
    m, atoms = QUERIES[case["query"]]
    st["query"] = q = gj.Query(ctx, m, atoms, less=LESS[case["query"]] if case.get("less") else ())
    if case["kind"] == "rows":
        cap = _rows_room(case)
        st["out"] = (np.zeros((cap, m), np.uint32) if case.get("host")
                     else torch.zeros((cap, m), dtype=torch.int32, device="cuda"))
    if case["kind"] == "update":
        st["there"], st["back"] = _update_batches(case, seed, src, dst)
        if case.get("rows"):  # the program's own copy of a batch's changes
            cap = _rows_room(case)
            st["changes"] = [(np.zeros((cap, m), np.uint32), np.zeros(cap, np.int8)) for _ in range(2)]
    return st


class _DeviceArray:
    """n 32-bit ids at a device address, for torch.as_tensor."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i4", "data": (ptr, False), "version": 2}


def _csr(g, n, edges):
    out = []
    for reverse in (False, True):
        ptrs = g.csr_ptrs(reverse)
        out.append([torch.as_tensor(_DeviceArray(p, k), device="cuda") if k else torch.empty(0, dtype=torch.int32)
                    for p, k in zip(ptrs, (n + 1, edges, edges))])
    return out


def _counters(s):
    return {k: s[k] for k in ("matches", "prefixes", "extensions")}


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "count":
        return _counters(gj.count(ctx, st["graph"], st["query"]))
    if kind == "rows":
        s, rows = gj.enumerate_rows(ctx, st["graph"], st["query"], out=st["out"])
        return {"stats": _counters(s), "rows": st["out"]}
    if kind == "batch":
        counts, stats = gj.run_batch(ctx, st["graph"], st["requests"])
        return {"counts": np.array(counts), "prefixes": np.array([s["prefixes"] for s in stats]),
                "extensions": np.array([s["extensions"] for s in stats])}
    if kind == "update":
        out = []
        want = case.get("rows", False)
        for i, (src, dst, sign) in enumerate((st["there"], st["back"])):
            cap = len(st["changes"][i][1]) if want else 0
            r = gj.apply_updates(ctx, st["graph"], src, dst, sign, [st["query"]], rows=want, cap=cap)[0]
            one = [r["count_delta"], [r["stats"][k] for k in ("prefixes", "extensions", "noop_inserts",
                                                              "noop_deletes", "raw_emissions")]]
            if want:
                rows, signs = st["changes"][i]
                rows[:r["n_delta"]] = r["rows"]
                signs[:r["n_delta"]] = r["signs"]
                one += [r["n_delta"], rows, signs]
            out.append(one)
        return out
    st["graph"] = None  # a program that loads its next graph has let the last one go
    st["graph"] = g = gj.Graph(ctx, st["src"], st["dst"], case["vertices"], **st["flags"])
    return _csr(g, case["vertices"], g.info(degrees=False)["edges"])


# ------------------------------------------------------- what a pass must do


def _distinct(case):
    """Edges left of the draws: R-MAT repeats thin out with the size."""
    if case["graph"] == "er":
        return case["draws"]
    return case["draws"] * (1.0 - 0.1835 * 0.687 ** ((math.log2(case["vertices"]) - 12) / 2))


def work(case):
    n, e = case["vertices"], _distinct(case)
    index = 4.0 * (n + 1) + 4.0 * e  # one direction, each entry once
    kind = case["kind"]
    if kind == "count":
        return {"bytes": index * (2 if case["query"] in ("cycle4", "cyclic_triangle") else 1), "flops": 0}
    if kind == "rows":
        # triangles of an R-MAT graph grow 2.207-fold a scale; 5.7e8 at 2^20 x 16
        t = 5.7e8 * 2.207 ** (math.log2(n) - 20) * (case["draws"] / (16.0 * n)) ** 2
        return {"bytes": index + 12.0 * t, "flops": 0}
    if kind == "batch":  # the slices' seed edges and the rows at both ends
        return {"bytes": case["requests"] * case["width"] / 4 * (8.0 + 2 * 4.0 * e / n), "flops": 0}
    if kind == "update":  # both batches in, the rows at both ends of a change read and written
        return {"bytes": 2.0 * case["size"] * (9.0 + 4 * 4.0 * e / n), "flops": 0}
    e = case["draws"] * (1 + 1 / 16)  # build: the list in, row pointers, columns and row ids out, both ways
    return {"bytes": 8.0 * case["draws"] * 1.125 + 2 * (4.0 * (n + 1) + 8.0 * e), "flops": 0}


def exact(case, seed):
    """Matches by dense 64-bit products where the adjacency matrix is small, and
    index arrays by sorting; None elsewhere."""
    if any(case.get(k) for k in ("degree_order", "undirected", "less")):
        return None
    n = case["vertices"]
    if case["kind"] == "build":
        src, dst = _edges(case, seed)
        k = _edge_set(src, dst, n)
        out = []
        for r, c in ((k // n, k % n), (k % n, k // n)):
            if out:
                r, c = (lambda t: (t // n, t % n))(torch.sort(r * n + c)[0])
            ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
            ptr[1:] = torch.bincount(r, minlength=n).cumsum(0)
            out.append([ptr.to(torch.int32), c.to(torch.int32), r.to(torch.int32)])
        return out
    if case["kind"] != "count" or n > 1 << 13 or case["query"] not in ("triangle", "cyclic_triangle", "diamond",
                                                                       "cycle4"):
        return None
    src, dst = _edges(case, seed)
    k = _edge_set(src, dst, n)
    a = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    a[k // n, k % n] = 1.0
    p = a @ a
    both = {"triangle": (p, a), "cyclic_triangle": (p, a.T), "diamond": (p, p), "cycle4": (p, p.T)}[case["query"]]
    return {"matches": int((both[0] * both[1]).sum().item()), "prefixes": None, "extensions": None}
