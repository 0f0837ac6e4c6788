"""The workloads that performance is judged on.

A case is a dict of plain values. `kind` names the entry point it goes through:

  solve     Context.solve / solve_async on a COO list (or the module's own solve)
  csr       Context.solve_csr_async on offsets and adjacency
  u64       Context.solve_u64_async on 8-byte IDs
  batch     Context.batch over many small graphs
  serve     Server.submit / wait over a burst of requests in host memory
  reducer   the steps of the distributed method on one device: every share of the
            entries solved into its own parent array, exported, packed, unpacked
            and merged by a Reducer

Graphs: `er` uniform endpoints; `rmat` R-MAT (0.57, 0.19, 0.19, 0.05) with the IDs
permuted; `extras` R-MAT followed by 1 % isolated IDs and short paths; `share` one
vertex range of a larger R-MAT graph, with the parent array of the whole graph;
`grid` a road-like square grid with streets missing, its IDs and entries in row order.
"""
import math

import numpy as np
import torch

import paper_2507_03695_amd as cc

DEV = "cuda"
CHUNK = 1 << 26          # entries generated at a time


# ---- sizes ----------------------------------------------------------------------------

def _path_lens(count):
    """Vertices of each appended path: 2..64."""
    return 2 + (np.arange(count, dtype=np.int64) * 37) % 63


def _graph_size(case):
    """(n, m): vertices and stored entries of the case's graph."""
    n, m = case["n"], case["m"]
    if case["graph"] == "extras":
        lens = _path_lens(case["paths"])
        n, m = n + n // 100 + int(lens.sum()), m + int((lens - 1).sum())
    if case.get("symmetric"):
        m *= 2
    return n, m


def _batch_sizes(case):
    """Vertices and entries of each graph: n log-uniform, mean degree uniform."""
    r = np.random.RandomState(case["G"] % 65521)
    lg = r.uniform(case["lg_lo"], case["lg_hi"], case["G"])
    ns = np.maximum(1, np.floor(2.0 ** lg)).astype(np.int64)
    ms = np.rint(ns * r.uniform(case["deg_lo"], case["deg_hi"], case["G"]) / 2).astype(np.int64)
    return ns, ms


def _serve_sizes(case):
    """Vertices and entries of each request: n from a Pareto(1.5) cut at 2^10 and
    2^24, 8 to 32 entries per vertex."""
    c = case["requests"]
    q = (np.arange(c) + 0.5) / c
    lo, hi = (2.0 ** 10) ** -1.5, (2.0 ** 24) ** -1.5
    ns = np.floor((lo - q * (lo - hi)) ** (-1 / 1.5)).astype(np.int64)
    r = np.random.RandomState(c % 65521)
    r.shuffle(ns)
    return ns, ns * r.randint(8, 33, c)


# ---- graphs ---------------------------------------------------------------------------

def _rmat_ids(scale, m, g):
    """The two endpoints (int64) of m R-MAT entries on 2^scale IDs, not permuted."""
    u = torch.zeros(m, dtype=torch.int32, device=DEV)
    v = torch.zeros(m, dtype=torch.int32, device=DEV)
    r = torch.empty(m, dtype=torch.float32, device=DEV)
    for _ in range(scale):
        r.uniform_(generator=g)
        down = r >= 0.76
        u.mul_(2).add_(down)
        v.mul_(2).add_(((r >= 0.57) & ~down) | (r >= 0.95))
    return u.long(), v.long()


def _coo(case, seed):
    """(edges (m, 2) int32 on the device, n)."""
    g = torch.Generator(device=DEV).manual_seed(seed * 1000003 + 17)
    kind, n0, m0 = case["graph"], case["n"], case["m"]
    n, m = _graph_size(case)
    e = torch.empty((m, 2), dtype=torch.int32, device=DEV)
    if kind == "grid":
        w = max(1, math.isqrt(n0))
        at = torch.randint(2 * n0, (m0,), generator=g, device=DEV).sort().values
        u = at // 2
        right = (u % w + 1 < w) & (u + 1 < n0)
        v = torch.where(at % 2 == 0, torch.where(right, u + 1, u), torch.where(u + w < n0, u + w, u))
        e[:m0, 0], e[:m0, 1] = u.int(), v.int()
    elif kind == "er":
        e[:m0].random_(0, n0, generator=g)
    else:
        scale = max(1, (n0 - 1).bit_length())
        perm = torch.randperm(n0, generator=g, device=DEV).int()
        # a share's first endpoints lie in one vertex range of the permuted IDs
        span = n0 // case["shares"] if kind == "share" else n0
        for at in range(0, m0, CHUNK):
            k = min(CHUNK, m0 - at)
            u, v = _rmat_ids(scale, k, g)
            u, v = perm[u % n0], perm[v % n0]
            e[at:at + k, 0], e[at:at + k, 1] = u % span, v
            del u, v
        if kind == "extras":
            lens = _path_lens(case["paths"])
            base = n0 + n0 // 100
            ids = np.arange(base, n)
            first = np.zeros(len(ids), bool)
            first[np.cumsum(lens) - lens] = True
            up = torch.from_numpy(ids[~first].astype(np.int32)).to(DEV).flip(0)
            tail = e[m0:m0 + up.numel()]
            tail[:, 0], tail[:, 1] = up, up - 1
    if case.get("symmetric"):
        h = m // 2
        e[h:, 0], e[h:, 1] = e[:h, 1], e[:h, 0]
    return e, n


def _csr(case, seed):
    e, n = _coo(case, seed)
    u, order = e[:, 0].sort(stable=True)
    adj = e[:, 1][order].contiguous()
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.bincount(u, minlength=n).cumsum(0)
    return off, adj, n


def _packed(ns, ms, seed):
    """Graphs of the given sizes with local IDs, even ones uniform and odd ones
    R-MAT, one after another: (vtx_off, edge_off, edges (sum m, 2) int32)."""
    g = torch.Generator(device=DEV).manual_seed(seed * 1000003 + 29)
    vo = np.concatenate([[0], np.cumsum(ns)])
    eo = np.concatenate([[0], np.cumsum(ms)])
    m = int(eo[-1])
    n_of = torch.from_numpy(ns).to(DEV)
    ends = torch.from_numpy(eo[1:]).to(DEV)
    bits = torch.ceil(torch.log2(n_of.double())).int()
    e = torch.empty((m, 2), dtype=torch.int32, device=DEV)
    top = int(bits.max())
    for at in range(0, m, CHUNK):
        k = min(CHUNK, m - at)
        of = torch.searchsorted(ends, torch.arange(at, at + k, device=DEV), right=True)
        n, b = n_of[of], bits[of]
        u = torch.zeros(k, dtype=torch.int32, device=DEV)
        v = torch.zeros(k, dtype=torch.int32, device=DEV)
        r = torch.empty(k, dtype=torch.float32, device=DEV)
        for level in range(top):
            r.uniform_(generator=g)
            on = b > level
            down = r >= 0.76
            u = torch.where(on, 2 * u + down, u)
            v = torch.where(on, 2 * v + (((r >= 0.57) & ~down) | (r >= 0.95)), v)
        rmat = of % 2 == 1
        for col, x in ((0, u), (1, v)):
            flat = (r.uniform_(generator=g).double() * n).long()
            skew = (x.long() % n * 1000003 + 12345) % n     # 1000003 is prime: a bijection
            e[at:at + k, col] = torch.minimum(torch.where(rmat, skew, flat), n - 1).int()
    return torch.from_numpy(vo).to(DEV), torch.from_numpy(eo).to(DEV), e


# ---- the cases ------------------------------------------------------------------------

def listed():
    return [
        # one request-sized graph, the smallest of the serving mix, through the one-line call
        {"name": "solve_small", "kind": "solve", "call": "module", "graph": "rmat", "n": 1500, "m": 12000,
         "zroot": False},
        # 65,536 vertices and 2^20 entries, whose parent array sits in any cache, labels waited for
        {"name": "solve_rmat_65k", "kind": "solve", "call": "sync", "graph": "rmat", "n": 65536,
         "m": 1 << 20, "zroot": False},
        # a mid-size skewed graph of no round size, with the zero root
        {"name": "solve_zroot_rmat_1m", "kind": "solve", "call": "async", "graph": "rmat", "n": 1000003,
         "m": 15000001, "zroot": True},
        # R-MAT scale 22 stored in both directions, declared symmetric
        {"name": "solve_rmat22_symmetric", "kind": "solve", "call": "async", "graph": "rmat", "n": 1 << 22,
         "m": 1 << 26, "zroot": False, "symmetric": True},
        # a large skewed graph by the default path, with isolated vertices and paths
        {"name": "solve_rmat25_extras", "kind": "solve", "call": "async", "graph": "extras", "n": 1 << 25,
         "m": 1 << 29, "paths": 5000, "zroot": False},
        # the headline: R-MAT scale 26 with isolated vertices and 10,000 paths, zero root
        {"name": "solve_zroot_rmat26_extras", "kind": "solve", "call": "async", "graph": "extras",
         "n": 1 << 26, "m": 1 << 30, "paths": 10000, "zroot": True},
        # one machine's sixteenth of R-MAT scale 28: a parent array far larger than any cache
        {"name": "solve_zroot_share28", "kind": "solve", "call": "async", "graph": "share", "n": 1 << 28,
         "m": 1 << 28, "shares": 16, "zroot": True},
        # a graph kept in CSR form, zero root from the row lengths
        {"name": "csr_zroot_rmat24", "kind": "csr", "graph": "extras", "n": 1 << 24, "m": 1 << 28,
         "paths": 3001, "zroot": True},
        # 8-byte vertex IDs
        {"name": "u64_rmat23", "kind": "u64", "graph": "rmat", "n": 1 << 23, "m": 1 << 27},
        # 4,096 graphs of 2^8 to 2^16 vertices in one launch
        {"name": "batch_4096", "kind": "batch", "G": 4096, "lg_lo": 8.0, "lg_hi": 16.0, "deg_lo": 2.0,
         "deg_hi": 32.0},
        # a burst of requests of all sizes from host memory
        {"name": "serve_1024", "kind": "serve", "requests": 1024},
        # eight shares of a skewed graph merged by a Reducer through compact IDs
        {"name": "reducer_rmat23_8", "kind": "reducer", "graph": "rmat", "n": (1 << 23) + 4099,
         "m": 120000001, "shares": 8},
    ]


def draw(rng):
    def log(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    def graph(n_lo, n_hi, m_hi, kinds):
        n = log(n_lo, n_hi)
        c = {"graph": rng.choice(kinds), "n": n}
        # uniform graphs stay below the density that joins every vertex
        ratio = rng.uniform(0.5, 0.3 * math.log(n) if c["graph"] == "er" else 24.0)
        c["m"] = max(1, min(int(n * ratio), m_hi))
        if c["graph"] == "extras":
            c["paths"] = rng.randint(1, max(2, n // 7000))
        if c["graph"] == "grid":
            c["m"] = max(1, min(int(2 * n * rng.uniform(0.4, 1.2)), m_hi))
        return c

    kind = rng.choice(["solve"] * 5 + ["csr"] * 2 + ["u64", "batch", "serve", "reducer"])
    if kind == "solve":
        c = dict(graph(1 << 8, 1 << 25, 1 << 28, ["er", "rmat", "extras", "grid"]), kind=kind,
                 call=rng.choice(["sync", "async"]), zroot=rng.random() < 0.5)
        if rng.random() < 0.2:
            c["symmetric"] = True
        return c
    if kind == "csr":
        c = dict(graph(1 << 10, 1 << 24, 1 << 27, ["er", "rmat", "extras", "grid"]), kind=kind,
                 zroot=rng.random() < 0.5)
        if rng.random() < 0.3:
            c["symmetric"] = True
        return c
    if kind == "u64":
        return dict(graph(1 << 10, 1 << 23, 1 << 26, ["er", "rmat", "extras", "grid"]), kind=kind)
    if kind == "batch":
        lo = rng.uniform(4.0, 12.0)
        return {"kind": kind, "G": log(8, 4096), "lg_lo": lo, "lg_hi": min(16.0, lo + rng.uniform(1.0, 6.0)),
                "deg_lo": rng.uniform(1.0, 4.0), "deg_hi": rng.uniform(6.0, 24.0)}
    if kind == "serve":
        return {"kind": kind, "requests": log(16, 1000)}
    return dict(graph(1 << 14, 1 << 22, 1 << 26, ["er", "rmat"]), kind=kind, shares=rng.choice([2, 4, 8, 16]))


# ---- preparation ----------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "serve":
        ns, ms = _serve_sizes(case)
        vo, eo, e = _packed(ns, ms, seed)
        e = np.ascontiguousarray(e.cpu().numpy()).view(np.uint32)
        vo, eo = vo.cpu().numpy(), eo.cpu().numpy()
        s["labels"] = np.empty(int(vo[-1]), np.uint32)
        s["requests"] = [(e[eo[i]:eo[i + 1]], int(ns[i]), s["labels"][vo[i]:vo[i + 1]])
                         for i in range(len(ns))]
        s["ctx"] = cc.Context(hbm_budget=8 << 30)
        s["server"] = cc.Server(s["ctx"], streams=4)
        return s
    s["ctx"] = cc.Context()
    if kind == "batch":
        ns, ms = _batch_sizes(case)
        s["vo"], s["eo"], s["edges"] = _packed(ns, ms, seed)
        s["L"] = torch.empty(int(ns.sum()), dtype=torch.int32, device=DEV)
        s["status"] = torch.empty(len(ns), dtype=torch.int32, device=DEV)
        return s
    s["flags"] = (cc.F_ZROOT if case.get("zroot") else 0) | (cc.F_SYMMETRIC if case.get("symmetric") else 0)
    if kind == "csr":
        s["off"], s["adj"], s["n"] = _csr(case, seed)
        s["L"] = torch.empty(s["n"], dtype=torch.int32, device=DEV)
        return s
    e, s["n"] = _coo(case, seed)
    if kind == "solve":
        s["edges"], s["call"] = e, case["call"]
        s["L"] = torch.empty(s["n"], dtype=torch.int32, device=DEV)
    elif kind == "u64":
        s["edges"] = e.long()
        s["L"] = torch.empty(s["n"], dtype=torch.int64, device=DEV)
    else:
        # each share holds the entries whose first endpoint lies in its vertex range;
        # the global zero root is agreed on beforehand
        g, n = case["shares"], s["n"]
        of = e[:, 0].long() * g // n
        s["parts"] = [e[of == k].contiguous() for k in range(g)]
        s["ctx"].zroot(e, n)
        s["z"] = s["ctx"].get_zroot()
        s["P"] = torch.empty(n, dtype=torch.int32, device=DEV)
        s["L"] = torch.empty(n, dtype=torch.int32, device=DEV)
    return s


# ---- one pass -------------------------------------------------------------------------

def _reduce(s):
    ctx, n, P, L, z = s["ctx"], s["n"], s["P"], s["L"], s["z"]
    hint = cc.F_ZROOT | cc.F_ZROOT_HINT
    pairs, zero = [], []
    for part in s["parts"]:
        ctx.init(n, P)
        ctx.zroot(part, n, flags=hint, zroot_hint=z)
        ctx.push(part, n, P)
        ctx.hook(part, n, P, flags=cc.F_ZROOT)
        ctx.compress(n, P, flags=cc.F_ZROOT)
        p, q = ctx.export_lists(P, n, z)
        pairs.append(p)
        zero.append(q)
    pairs, zero = torch.cat(pairs), torch.cat(zero)
    k = ctx.id_bytes(n)
    wire_p, wire_z = ctx.pack_ids(pairs, k), ctx.pack_ids(zero, k)
    pairs = ctx.unpack_ids(wire_p, pairs.numel(), k).view(-1, 2)
    zero = ctx.unpack_ids(wire_z, zero.numel(), k)
    ctx.init(n, L)
    ctx.zroot(pairs, n, flags=hint, zroot_hint=z)
    ctx.hook(pairs, n, L, flags=cc.F_ZROOT)
    ctx.hook_ids(zero, z, n, L, flags=cc.F_ZROOT)
    ctx.compress(n, L, flags=cc.F_ZROOT)
    ctx.canon(n, L)
    return L


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "solve":
        if s["call"] == "module":
            return cc.solve(s["edges"], s["n"])
        if s["call"] == "sync":
            return ctx.solve(s["edges"], s["n"], flags=s["flags"])
        ctx.solve_async(s["edges"], s["n"], s["L"], flags=s["flags"])
        return s["L"]
    if kind == "csr":
        ctx.solve_csr_async(s["off"], s["adj"], s["n"], s["L"], flags=s["flags"])
        return s["L"]
    if kind == "u64":
        ctx.solve_u64_async(s["edges"], s["n"], s["L"])
        return s["L"]
    if kind == "batch":
        L, status = ctx.batch(s["vo"], s["eo"], s["edges"], s["L"], s["status"])
        return {"labels": L, "status": status}
    if kind == "serve":
        tickets = [s["server"].submit(e, n, L) for e, n, L in s["requests"]]
        codes = [s["server"].wait(t)[0] for t in tickets]
        return {"labels": s["labels"], "status": np.array(codes, np.int32)}
    return _reduce(s)


# ---- what a pass cannot do without ------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        ns, ms = _batch_sizes(case) if kind == "batch" else _serve_sizes(case)
        return {"bytes": 8 * int(ms.sum()) + 4 * int(ns.sum()) + 20 * len(ns), "flops": 0}
    n, m = _graph_size(case)
    if kind == "csr":
        return {"bytes": 4 * m + 8 * (n + 1) + 4 * n, "flops": 0}
    if kind == "u64":
        return {"bytes": 16 * m + 8 * n, "flops": 0}
    return {"bytes": 8 * m + 4 * n, "flops": 0}


# ---- the labels by another road ---------------------------------------------------------

def _min_labels(u, v, n):
    """Smallest ID of every vertex's component, by repeated minima over the entries."""
    dev = u.device
    L = torch.arange(n, device=dev)
    while True:
        moved = False
        for at in range(0, u.numel(), CHUNK):
            a, b = L[u[at:at + CHUNK].long()], L[v[at:at + CHUNK].long()]
            lo, hi = torch.minimum(a, b), torch.maximum(a, b)
            on = lo < hi
            if bool(on.any()):
                moved = True
                L.scatter_reduce_(0, hi[on], lo[on], "amin")
            del a, b, lo, hi, on
        if not moved:
            return L
        while True:
            up = L[L]
            if bool((up == L).all()):
                break
            L = up


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        ns, ms = _batch_sizes(case) if kind == "batch" else _serve_sizes(case)
        vo, eo, e = _packed(ns, ms, seed)
        of = torch.repeat_interleave(torch.arange(len(ns), device=DEV), torch.from_numpy(ms).to(DEV))
        base = vo[:-1][of]
        L = _min_labels(e[:, 0] + base, e[:, 1] + base, int(vo[-1]))
        L -= torch.repeat_interleave(vo[:-1], torch.from_numpy(ns).to(DEV))
        status = np.zeros(len(ns), np.int32)
        if kind == "serve":
            return {"labels": L.int().cpu().numpy().view(np.uint32), "status": status}
        return {"labels": L.int(), "status": torch.from_numpy(status)}
    e, n = _coo(case, seed)
    L = _min_labels(e[:, 0], e[:, 1], n)
    return L if kind == "u64" else L.int()
