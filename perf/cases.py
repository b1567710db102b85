"""The work that programs have this library do, case by case, through its public entry points.

Every case is a call (or a load followed by a call) on synthetic graphs of the families the library is
benchmarked and tested on: R-MAT graphs for cliques and small motifs, labelled and unlabelled G(n, m) graphs for
frequent subgraphs and 5-motifs, and batches of small G(n, p) graphs.  A graph is made on the GPU from the seed
alone and handed over as device arrays.  All results are whole numbers (counts, supports, vertex ids), so there is
no 64-bit reference to compare them with: they have to be equal.
"""
import math

import numpy as np
import torch

from paper_1911_06969_amd import binding, synth


# ------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 2654435761 % (1 << 62))


def _rmat_pairs(n, ef, gen, a=0.57, b=0.19, c=0.19):
    """About ef * n directed R-MAT pairs over n vertices (the recursion runs on the next power of two and
    pairs outside [0, n) are dropped), under a random renaming of the vertices."""
    m = int(ef * n)
    u = torch.zeros(m, dtype=torch.int64, device="cuda")
    v = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(max(1, (n - 1).bit_length())):
        r = torch.rand(m, generator=gen, device="cuda")
        u = 2 * u + (r >= a + b)
        v = 2 * v + (((r >= a) & (r < a + b)) | (r >= a + b + c))
    keep = (u < n) & (v < n)
    name = torch.randperm(n, generator=gen, device="cuda")
    return name[u[keep]], name[v[keep]]


def _uniform_pairs(n, degree, gen):
    m = int(n * degree / 2)
    return (torch.randint(0, n, (m,), generator=gen, device="cuda"),
            torch.randint(0, n, (m,), generator=gen, device="cuda"))


def _rows(n, src):
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=row_ptr[1:])
    return row_ptr


def _canonical(n, u, v):
    """Symmetric, loop-free, duplicate-free CSR with ascending rows."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    src = key // n
    return _rows(n, src), (key - src * n).to(torch.int32)


def _as_read(n, u, v):
    """The pairs as an edge list sorted by source only: one direction, with loops, repeats and unordered rows."""
    u, order = torch.sort(u, stable=True)
    return _rows(n, u), v[order].to(torch.int32)


def _pairs(case, gen):
    if case["graph"] == "rmat":
        return _rmat_pairs(case["n"], case["ef"], gen)
    return _uniform_pairs(case["n"], case["degree"], gen)


def _graph(case, gen):
    n = case["n"]
    row_ptr, col = _canonical(n, *_pairs(case, gen))
    labels = None
    if case.get("labels"):
        labels = torch.randint(0, case["labels"], (n,), generator=gen, device="cuda", dtype=torch.int32)
    return binding.Graph(row_ptr, col, labels, case.get("labels", 0), stream=torch.cuda.current_stream())


def _batch(case, seed):
    b = synth.er_batch(case["graphs"], case["n_min"], case["n_max"], case["p_min"], case["p_max"], seed=int(seed) + 1)
    return b, binding.pg_batch_load(b.voff, b.row_ptr, b.col, stream=torch.cuda.current_stream())


class _Slot:
    """A loaded batch and one asynchronous slot on it, released together."""

    def __init__(self, batch, max_ids):
        self.batch = batch
        self.slot = binding.pg_batch_slot_create(batch, max_ids)

    def __del__(self):
        binding.pg_batch_slot_free(self.slot)
        binding.pg_batch_free(self.batch)


class _Batch:
    def __init__(self, handle):
        self.h = handle

    def __del__(self):
        binding.pg_batch_free(self.h)


# ------------------------------------------------------------------- cases

def listed():
    return [
        # Triangle counting on a small graph: one short call, as an interactive query makes it.
        {"name": "tc_rmat14", "do": "cliques", "graph": "rmat", "n": 1 << 14, "ef": 8, "k": 3},
        # The headline: 4-cliques of a Patents-sized skewed graph.
        {"name": "clique4_rmat21", "do": "cliques", "graph": "rmat", "n": 1 << 21, "ef": 13, "k": 4},
        # Deeper cliques, where the work is no longer in finding triangles; a vertex count off any power of two.
        {"name": "clique5_rmat20", "do": "cliques", "graph": "rmat", "n": 1_000_003, "ef": 10, "k": 5},
        # Clique listing: the rows themselves are wanted, for a caller's array of a fixed number of rows.
        {"name": "list3_rmat14", "do": "list", "graph": "rmat", "n": 1 << 14, "ef": 8, "k": 3, "capacity": 1 << 19},
        # Motif counting on a Mico-sized skewed graph, three and four vertices.
        {"name": "motif3_rmat18", "do": "motifs", "graph": "rmat", "n": 1 << 18, "ef": 8, "k": 3},
        {"name": "motif4_rmat18", "do": "motifs", "graph": "rmat", "n": 1 << 18, "ef": 8, "k": 4},
        # Five-vertex motifs on a sparse uniform graph.
        {"name": "motif5_er100k", "do": "motifs", "graph": "uniform", "n": 100_000, "degree": 8.0, "k": 5},
        # Frequent patterns of up to two edges on a Mico-sized labelled graph.
        {"name": "fsm2_er100k", "do": "fsm", "graph": "uniform", "n": 100_000, "degree": 21.6, "labels": 29,
         "edges": 2, "support": 300},
        # Frequent patterns of up to three edges on the large labelled graph.
        {"name": "fsm3_er500k", "do": "fsm", "graph": "uniform", "n": 500_000, "degree": 8.0, "labels": 16,
         "edges": 3, "support": 1000},
        # Many small graphs in one call (offline scoring of a collection).
        {"name": "batch4_10k", "do": "batch", "graphs": 10_000, "n_min": 10, "n_max": 400, "p_min": 0.02,
         "p_max": 0.3, "k": 4},
        # One micro-batch of a serving loop: submitted to an asynchronous slot and waited for.
        {"name": "serve4_64", "do": "serve", "graphs": 2_000, "n_min": 10, "n_max": 400, "p_min": 0.02, "p_max": 0.3,
         "k": 4, "ids": 64, "max_ids": 1024},
        # A graph that is counted once: raw edges in, canonicalised, validated, oriented, triangles out, released.
        {"name": "load3_rmat18", "do": "load", "graph": "rmat", "n": 1 << 18, "ef": 8, "k": 3, "raw": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["cliques", "cliques", "list", "motif3", "motif4", "motif5", "fsm", "fsm", "batch", "serve", "load"])
    if do == "cliques":
        k = rng.choice([3, 4, 4, 5, 6])
        n = _log_int(rng, 1 << 10, {3: 1 << 21, 4: 1 << 21, 5: 1 << 20, 6: 1 << 15}[k])
        return {"do": "cliques", "graph": "rmat", "n": n, "ef": rng.randint(4, 13 if k < 5 else 10), "k": k}
    if do == "list":
        return {"do": "list", "graph": "rmat", "n": _log_int(rng, 1 << 9, 1 << 16), "ef": rng.randint(4, 10),
                "k": rng.choice([2, 3, 4]), "capacity": _log_int(rng, 1 << 10, 1 << 20)}
    if do == "motif3":
        return {"do": "motifs", "graph": "rmat", "n": _log_int(rng, 1 << 10, 1 << 19), "ef": rng.randint(4, 12), "k": 3}
    if do == "motif4":
        return {"do": "motifs", "graph": "rmat", "n": _log_int(rng, 1 << 10, 1 << 18), "ef": rng.randint(3, 8), "k": 4}
    if do == "motif5":
        return {"do": "motifs", "graph": "uniform", "n": _log_int(rng, 1000, 100_000),
                "degree": round(rng.uniform(3.0, 10.0), 2), "k": 5}
    if do == "fsm":
        edges = rng.choice([1, 2, 2, 3, 3, 4])
        n = _log_int(rng, 2000, {1: 500_000, 2: 200_000, 3: 500_000, 4: 20_000}[edges])
        return {"do": "fsm", "graph": "uniform", "n": n, "degree": round(rng.uniform(4.0, 20.0 if edges < 3 else 8.0), 2),
                "labels": rng.randint(4, 29 if edges < 4 else 12), "edges": edges,
                "support": max(2, int(n * rng.uniform(0.0005, 0.01)))}
    if do in ("batch", "serve"):
        n_max = _log_int(rng, 24, 500)
        case = {"do": do, "graphs": _log_int(rng, 200, 8000 if n_max <= 400 else 3000), "n_min": rng.randint(4, 20),
                "n_max": n_max, "p_min": 0.02, "p_max": round(rng.uniform(0.1, 0.35), 3), "k": rng.choice([3, 4, 4])}
        if do == "serve":
            case["graphs"] = min(case["graphs"], 2000)
            case["ids"], case["max_ids"] = _log_int(rng, 1, 1024), 1024
        return case
    return {"do": "load", "graph": "rmat", "n": _log_int(rng, 1 << 12, 1 << 20), "ef": rng.randint(4, 12),
            "k": rng.choice([3, 4]), "raw": rng.random() < 0.7}


def prepare(case, seed):
    gen = _generator(seed)
    do = case["do"]
    if do in ("cliques", "motifs", "fsm", "list"):
        return {"case": case, "graph": _graph(case, gen)}
    if do == "load":
        u, v = _pairs(case, gen)
        row_ptr, col = _as_read(case["n"], u, v) if case["raw"] else _canonical(case["n"], u, v)
        return {"case": case, "row_ptr": row_ptr, "col": col}
    b, handle = _batch(case, seed)
    if do == "batch":
        return {"case": case, "batch": _Batch(handle)}
    ids = np.random.default_rng(int(seed)).choice(b.n_graphs, case["ids"], replace=True).astype(np.int64)
    return {"case": case, "slot": _Slot(handle, case["max_ids"]), "ids": ids}


def run(state):
    case = state["case"]
    do, k = case["do"], case.get("k")
    if do == "cliques":
        return state["graph"].cliques(k)
    if do == "list":
        rows, total = state["graph"].list_cliques(k, case["capacity"])
        return {"rows": rows, "total": total}
    if do == "motifs":
        return state["graph"].motifs(k)
    if do == "fsm":
        supports, frequent = state["graph"].fsm(case["edges"], case["support"])
        return {"supports": supports, "frequent": frequent}
    if do == "batch":
        return binding.pg_batch_count_motifs(state["batch"].h, k, None, n_graphs=case["graphs"])
    if do == "serve":
        slot = state["slot"].slot
        return binding.pg_batch_slot_wait(slot, binding.pg_batch_slot_submit(slot, k, state["ids"]), k)
    with binding.Graph(state["row_ptr"], state["col"], stream=torch.cuda.current_stream(),
                       canonicalize=case["raw"]) as g:
        n, nnz, max_degree = g.info()
        return {"n": n, "entries": nnz, "max_degree": max_degree, "cliques": g.cliques(k)}


def work(case):
    """Bytes of the graph read once and of the results written once.  The work is whole-number set intersection,
    whose least amount depends on the graph, so no operations are claimed."""
    if case["do"] in ("batch", "serve"):
        n, p = (case["n_min"] + case["n_max"]) / 2, (case["p_min"] + case["p_max"]) / 2
        square = (case["n_max"] ** 2 + case["n_max"] * case["n_min"] + case["n_min"] ** 2) / 3
        graphs = case["graphs"] if case["do"] == "batch" else case["ids"]
        return {"bytes": graphs * (8 * n + 4 * p * square + (48 if case["k"] == 4 else 16)), "flops": 0}
    n = case["n"]
    entries = 2 * n * case["ef"] if case["graph"] == "rmat" else n * case["degree"]
    nbytes = 8 * (n + 1) + 4 * entries
    if case["do"] == "load" and case["raw"]:
        nbytes -= 2 * entries   # one direction only
    if case["do"] == "list":
        nbytes += 4 * case["k"] * case["capacity"]
    if case["do"] == "fsm":
        nbytes += 4 * n + 8 * binding.pg_fsm_num_patterns(case["edges"], case["labels"])
    return {"bytes": nbytes, "flops": 0}
