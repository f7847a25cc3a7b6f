"""The workloads whose speed is followed: one pass of each goes through the public entry points
of the package as a program that solves vertex-cover problems calls them.

Every case names a kind (how graphs are drawn and which entry point solves them) and its sizes.
All graphs are drawn from the seed alone. Outputs are what does not depend on the schedule of
the parallel search: sizes and decisions always; covers where the reduction rules settle a graph
at its root; node counts where the answer is no (the whole tree is visited). The search of a
minimum or of a yes-answer may find any one of several covers, so those covers are not returned.
"""

import functools
import math
import types

import numpy as np
import torch

import paper_2204_10402_amd as vc

DEVICE = "cuda:0"


# ---- graphs ------------------------------------------------------------------------------------

def _csr(n, u, v):
    """Sorted symmetric CSR of the distinct loop-free pairs among (u, v)."""
    u, v = np.asarray(u, np.int64), np.asarray(v, np.int64)
    lo, hi = np.minimum(u, v), np.maximum(u, v)
    key = np.unique((lo * n + hi)[lo != hi])
    lo, hi = key // n, key % n
    both = np.sort(np.concatenate([key, hi * n + lo]))
    row_ptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(both // n, minlength=n), out=row_ptr[1:])
    return types.SimpleNamespace(n=n, row_ptr=row_ptr, col_idx=(both % n).astype(np.int32))


def _er(rng, n, degree):
    """G(n, p) with p = degree / n; sparse ones by drawing the number of edges, then the edges."""
    p = min(1.0, degree / n)
    if n <= 1024:
        iu, ju = np.triu_indices(n, 1)
        keep = rng.random(iu.size) < p
        return _csr(n, iu[keep], ju[keep])
    m = rng.binomial(n * (n - 1) // 2, p)
    return _csr(n, rng.integers(0, n, m), rng.integers(0, n, m))


def _regular(rng, n, d):
    """Random d-regular graph by the configuration model (whole pairing redrawn on a clash)."""
    stubs = np.repeat(np.arange(n, dtype=np.int64), d)
    while True:
        pairs = rng.permutation(stubs).reshape(-1, 2)
        lo, hi = pairs.min(1), pairs.max(1)
        if np.all(lo != hi) and np.unique(lo * n + hi).size == lo.size:
            return _csr(n, lo, hi)


def _planted(rng, n, c, m):
    """Hidden cover of c vertices: about m edges, three quarters from it to the rest, a quarter
    inside it (repeated pairs and loops drop out)."""
    perm = rng.permutation(n)
    cover, rest = perm[:c], perm[c:]
    cross = int(round(0.75 * m))
    u = cover[rng.integers(0, c, m)]
    v = np.concatenate([rest[rng.integers(0, n - c, cross)], cover[rng.integers(0, c, m - cross)]])
    return _csr(n, u, v)


def _planted_many(rng, count, n_lo, n_hi):
    """`count` planted graphs of n_lo..n_hi vertices, average degree 3..12 and a hidden cover of
    0.3 n, drawn all at once and packed: (n, nnz, row_ptr, col_idx, cover sizes)."""
    n = rng.integers(n_lo, n_hi + 1, count)
    c = (0.3 * n).astype(np.int64)
    m = np.round(rng.uniform(3, 12, count) * n / 2).astype(np.int64)
    cross = np.round(0.75 * m).astype(np.int64)
    inst = np.repeat(np.arange(count), m)
    within = np.arange(inst.size) - np.repeat(np.cumsum(m) - m, m)
    to_rest = within < cross[inst]
    # vertices are numbered by a multiplier coprime to n, so that the cover is spread over the ids
    step = 1 + 2 * (n // 5)
    while np.any(bad := np.gcd(step, n) != 1):
        step[bad] += 1
    draw = lambda size: (rng.random(inst.size) * size).astype(np.int64)  # noqa: E731
    place = lambda x: x * step[inst] % n[inst]  # noqa: E731
    u = place(draw(c[inst]))
    v = place(np.where(to_rest, c[inst] + draw(n[inst] - c[inst]), draw(c[inst])))
    base = (np.cumsum(n) - n)[inst]
    total = int(n.sum())
    lo, hi = np.minimum(u, v) + base, np.maximum(u, v) + base
    key = np.unique((lo * total + hi)[lo != hi])
    both = np.sort(np.concatenate([key, key % total * total + key // total]))
    src, dst = both // total, both % total
    degree = np.bincount(src, minlength=total)
    owner = np.repeat(np.arange(count), n)
    first = np.cumsum(n) - n
    nnz = np.bincount(owner, weights=degree, minlength=count).astype(np.int64)
    ends = np.cumsum(degree) - np.repeat(np.cumsum(nnz) - nnz, n)
    row_ptr = np.zeros(total + count, np.int32)
    row_ptr[np.arange(total) + owner + 1] = ends
    col_idx = (dst - first[owner[src]]).astype(np.int32)
    return n.astype(np.int32), nnz.astype(np.int32), row_ptr, col_idx, c.astype(np.int32)


# ---- handles a program keeps -------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _solver():
    return vc.Solver(0)


@functools.lru_cache(maxsize=None)
def _server():
    return vc.Server(0)


def _on_device(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE)


def _packed(graphs):
    n, nnz, rp, ci = vc.pack_batch(graphs)
    return n, nnz, _on_device(rp), _on_device(ci)


def _tau(graphs):
    """Minimum cover sizes: what a program knows that then asks for the proof that one vertex
    fewer is not enough."""
    return _solver().mvc_batch_device(*_packed(graphs)).size.astype(np.int32)


# ---- the cases ---------------------------------------------------------------------------------

def listed():
    return [
        # Smallest calls: a program that solves graphs of 60 vertices one call at a time. Launches
        # and the chain of a few dozen dependent nodes are all there is.
        {"name": "small-mvc-calls", "kind": "mvc-calls", "n": 60, "degree": 6.0, "count": 8},
        # The same from code that brings its own device workspace and asks for a decision.
        {"name": "small-pvc-ws-calls", "kind": "pvc-ws-calls", "n": 190, "degree": 8.0, "count": 8},
        # The exhaustive searches of the benchmark, one batched call with the autotuner.
        {"name": "hard-mvc-batch", "kind": "mvc-batch", "regular": 120, "er": 150, "count": 16},
        # One hard graph alone: the proof that k = minimum - 1 is not enough.
        {"name": "hard-pvc-no", "kind": "pvc-no", "family": "regular", "n": 120, "degree": 5.0,
         "count": 1},
        # The same on dense graphs, the paper's other class, with the widest bitsets.
        {"name": "dense-pvc-no", "kind": "pvc-no", "family": "er", "n": 200, "degree": 100.0,
         "count": 1},
        # Deep searches above the bitset sizes (degree arrays), a few graphs in one call.
        {"name": "array-pvc-no", "kind": "pvc-no", "family": "er", "n": 390, "degree": 3.5,
         "count": 16},
        # A few graphs of thousands of vertices whose reduction at the root settles them.
        {"name": "planted-pvc-batch", "kind": "planted", "n": 5000, "cover": 400, "edges": 40000,
         "count": 8},
        # One large graph, and one whose node does not fit beside a workgroup's other memory.
        {"name": "planted-pvc-large", "kind": "planted", "n": 16000, "cover": 800,
         "edges": 128000, "count": 1},
        {"name": "planted-pvc-huge", "kind": "planted", "n": 50021, "cover": 500, "edges": 100000,
         "count": 1},
        # Throughput: thousands of small instances in one call, both kernel families.
        {"name": "planted-small-batch", "kind": "planted-many", "n_lo": 40, "n_hi": 400,
         "count": 4096},
        # A sparse network from host memory: greedy bound, reductions and a small search.
        {"name": "sparse-mvc-host", "kind": "mvc-host", "n": 5000, "degree": 2.5},
        # A stream of mixed requests through the server.
        {"name": "served-stream", "kind": "served", "n_lo": 50, "n_hi": 2000, "count": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mvc-calls", "pvc-ws-calls", "mvc-batch", "pvc-no", "dense", "array",
                       "planted", "planted-many", "mvc-host", "served"])
    if kind == "mvc-calls":
        return {"kind": kind, "n": rng.randint(20, 90), "degree": round(rng.uniform(3, 8), 2),
                "count": rng.randint(4, 8)}
    if kind == "pvc-ws-calls":
        return {"kind": kind, "n": _log_int(rng, 40, 600), "degree": round(rng.uniform(4, 8), 2),
                "count": rng.randint(4, 8)}
    if kind == "mvc-batch":
        return {"kind": kind, "regular": 2 * rng.randint(40, 58), "er": rng.randint(90, 140),
                "count": rng.randint(4, 16)}
    if kind == "pvc-no":
        family = rng.choice(["regular", "er"])
        return {"kind": kind, "family": family, "n": 2 * rng.randint(30, 57),
                "degree": float(rng.randint(3, 5)) if family == "regular"
                else round(rng.uniform(4, 11), 2), "count": rng.randint(1, 3)}
    if kind == "dense":
        n = rng.randint(70, 200)
        return {"kind": "pvc-no", "family": "er", "n": n,
                "degree": round(n * rng.uniform(0.5, 0.8), 2), "count": rng.randint(1, 2)}
    if kind == "array":
        return {"kind": "pvc-no", "family": "er", "n": rng.randint(257, 380),
                "degree": round(rng.uniform(2.8, 3.4), 2), "count": rng.randint(4, 16)}
    if kind == "planted":
        n = _log_int(rng, 3000, 18000)
        return {"kind": kind, "n": n, "cover": n * rng.randint(5, 9) // 100,
                "edges": n * rng.randint(6, 8), "count": rng.randint(1, 8) if n <= 6000 else 1}
    if kind == "planted-many":
        n_lo = rng.randint(30, 100)
        return {"kind": kind, "n_lo": n_lo, "n_hi": n_lo + rng.randint(50, 300),
                "count": _log_int(rng, 128, 4096)}
    if kind == "mvc-host":
        return {"kind": kind, "n": _log_int(rng, 400, 5000), "degree": round(rng.uniform(1.8, 2.5), 2)}
    return {"kind": kind, "n_lo": 50, "n_hi": rng.randint(300, 2000), "count": _log_int(rng, 32, 256)}


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "mvc-calls":
        graphs = [_er(rng, case["n"], case["degree"]) for _ in range(case["count"])]
        s["graphs"] = [(_on_device(g.row_ptr), _on_device(g.col_idx)) for g in graphs]
        _solver()
    elif kind == "pvc-ws-calls":
        n, c = case["n"], int(0.3 * case["n"])
        graphs = [_planted(rng, n, c, int(round(case["degree"] * n / 2)))
                  for _ in range(case["count"])]
        s["graphs"] = [(_on_device(g.row_ptr), _on_device(g.col_idx),
                        torch.zeros(n, dtype=torch.uint8, device=DEVICE),
                        c - int(rng.integers(0, 2))) for g in graphs]
        most = max(_solver().workspace_bytes(n, g.col_idx.size, depth=c + 1) for g in graphs)
        s["workspace"] = torch.empty(most, dtype=torch.uint8, device=DEVICE)
    elif kind == "mvc-batch":
        half = case["count"] // 2
        s["batch"] = _packed([_regular(rng, case["regular"], 5) for _ in range(case["count"] - half)] +
                             [_er(rng, case["er"], 0.08 * case["er"]) for _ in range(half)])
        s["options"] = vc.Options(flags=vc.OPT_AUTOTUNE)
        _solver()
    elif kind == "pvc-no":
        graphs = [_regular(rng, case["n"], int(case["degree"])) if case["family"] == "regular"
                  else _er(rng, case["n"], case["degree"]) for _ in range(case["count"])]
        s["k"] = _tau(graphs) - 1
        s["batch"] = _packed(graphs)
        s["cover"] = torch.zeros(int(s["batch"][0].sum()), dtype=torch.uint8, device=DEVICE)
    elif kind == "planted":
        s["batch"] = _packed([_planted(rng, case["n"], case["cover"], case["edges"])
                              for _ in range(case["count"])])
        # the hidden cover's size, and (every second graph) one less
        s["k"] = case["cover"] - (np.arange(case["count"], dtype=np.int32) % 2)
        s["cover"] = torch.zeros(case["n"] * case["count"], dtype=torch.uint8, device=DEVICE)
        _solver()
    elif kind == "planted-many":
        n, nnz, rp, ci, c = _planted_many(rng, case["count"], case["n_lo"], case["n_hi"])
        s["batch"] = n, nnz, _on_device(rp), _on_device(ci)
        s["k"] = c - rng.integers(0, 2, case["count"]).astype(np.int32)
        s["cover"] = torch.zeros(int(n.sum()), dtype=torch.uint8, device=DEVICE)
        _solver()
    elif kind == "mvc-host":
        s["graph"] = _er(rng, case["n"], case["degree"])
        _solver()
    else:
        s["requests"] = requests = []
        for _ in range(case["count"]):
            if rng.random() < 0.6:
                n = int(round(math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"])))))
                c = int(0.3 * n)
                g = _planted(rng, n, c, int(round(rng.uniform(3, 8) * n / 2)))
                requests.append((g, "pvc", c - int(rng.integers(0, 2))))
            else:
                n = 2 * int(rng.integers(25, 40))
                g = _regular(rng, n, 3) if rng.random() < 0.3 else _er(rng, n, rng.uniform(4, 8))
                requests.append((g, "mvc", 0))
        _server()
    return s


def run(s):
    kind = s["kind"]
    if kind == "mvc-calls":
        out = [_solver().mvc_device(rp, ci) for rp, ci in s["graphs"]]
        return {"size": np.array([r.size for r in out], np.int32),
                "greedy": np.array([r.stats["greedy_size"] for r in out], np.int32)}
    if kind == "pvc-ws-calls":
        out = [_solver().pvc_device_ws(rp, ci, k, s["workspace"], cover)
               for rp, ci, cover, k in s["graphs"]]
        return {"yes": np.array([r.yes for r in out], np.int32),
                "size": np.array([r.size for r in out], np.int32),
                "cover": [g[2] for g in s["graphs"]]}
    if kind == "mvc-batch":
        r = _solver().mvc_batch_device(*s["batch"], options=s["options"])
        return {"status": r.status, "size": r.size}
    if kind == "pvc-no":
        r = _solver().pvc_batch_device(*s["batch"], s["k"], s["cover"])
        return {"status": r.status, "yes": r.yes, "size": r.size, "nodes": r.nodes, "cover": r.cover}
    if kind == "planted":
        r = _solver().pvc_batch_device(*s["batch"], s["k"], s["cover"])
        return {"status": r.status, "yes": r.yes, "size": r.size, "nodes": r.nodes, "cover": r.cover}
    if kind == "planted-many":
        r = _solver().pvc_batch_device(*s["batch"], s["k"], s["cover"])
        return {"status": r.status, "yes": r.yes, "nodes_of_no": np.where(r.yes, 0, r.nodes)}
    if kind == "mvc-host":
        r = _solver().mvc(s["graph"])
        return {"size": r.size, "greedy": r.stats["greedy_size"]}
    server, place, done = _server(), {}, 0
    for i, (g, problem, k) in enumerate(s["requests"]):
        place[server.submit(g, problem, k)] = i
    size = np.zeros(len(place), np.int32)
    yes = np.zeros(len(place), np.int32)
    while done < len(place):
        for r in server.poll(timeout_ms=1000):
            size[place[r["ticket"]]] = r["size"]
            yes[place[r["ticket"]]] = r["yes"]
            done += 1
    return {"size": size, "yes": yes}


def work(case):
    """Bytes: each CSR read once (4 bytes per row pointer and entry), one byte per vertex of the
    cover written where a pass asks for it. Operations: of a search, only what every node has to
    do at least, one test per vertex of its graph, at a typical number of nodes; of a graph
    settled at the root, one per entry."""
    kind, count = case["kind"], case.get("count", 1)
    if kind == "mvc-batch":
        half = count // 2
        n = (case["regular"] * (count - half) + case["er"] * half) / count
        entries = (5 * case["regular"] * (count - half) + 0.08 * case["er"] ** 2 * half) / count
        nodes = 5e6 * 2 ** ((n - 135) / 6)
    elif kind == "planted":
        n, entries, nodes = case["n"], 2 * case["edges"], 1
    elif kind == "planted-many":
        n = (case["n_lo"] + case["n_hi"]) / 2
        entries, nodes = 7.5 * n, 3
    elif kind == "served":
        n = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        entries, nodes = 5.5 * n, 5
    else:
        n, entries = case["n"], case["n"] * case["degree"]
        nodes = {"mvc-calls": 30, "pvc-ws-calls": 2, "mvc-host": 5, "pvc-no": 1e4}[kind]
    cover = n if kind in ("pvc-ws-calls", "pvc-no", "planted", "planted-many", "mvc-host", "served") else 0
    return {"bytes": float(count * (4 * (n + 1 + entries) + cover)),
            "flops": float(count * (nodes * n + entries))}


def exact(case, seed):
    """Every output is a whole number or a byte, which stays the same: nothing is rounded."""
    return None
