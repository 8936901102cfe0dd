"""Timed work of the library's users: PageRank and Graph SGD side tasks, and the GEMM load of the stage beside them.

A case is a dict of plain values; `kind` says which path of the library it takes:
  pagerank   fr_pagerank_run_standalone on a task whose layout exists: `iterations` passes over the graph, as every
             run of a task after its first
  new_graph  a graph the library has not seen: task made, layout built, `iterations` passes, task destroyed
  harvest    the life of a side task in a stage's bubbles: registered, initialised in one bubble, run in the next,
             stopped
  sgd        fr_sgd_run_standalone: `iterations` passes over a rating graph, factors updated in place
  load       one forward and one backward burst of the stage load (fr_load_fp, fr_load_bp)
  gemm       one fr_gemm_bf16
Inputs are made on the GPU from the seed: R-MAT (.57, .19, .19, .05) or fixed out-degree edges over any number of
vertices, ids scattered by a random permutation; ratings of planted low-rank factors plus noise; uniform GEMM operands.
"""
import math
import time

import torch

import paper_2409_06941_amd as fr

DAMPING = 0.85
GAMMA, LAMBDA = 0.01, 0.02


def listed():
    return [
        # the smallest configuration's graph: two launches of a few microseconds per iteration
        dict(name="pagerank_tiny", kind="pagerank", graph="rmat", vertices=1 << 14, edges=1 << 18, iterations=30, cus=0),
        # a graph whose sizes are no multiples of anything, fewer edges per vertex
        dict(name="pagerank_ragged", kind="pagerank", graph="rmat", vertices=1_000_003, edges=9_999_991, iterations=20, cus=0),
        # three of the benchmark's skewed graphs, up to its headline configuration
        dict(name="pagerank_medium", kind="pagerank", graph="rmat", vertices=1 << 22, edges=1 << 26, iterations=50, cus=0),
        dict(name="pagerank_large", kind="pagerank", graph="rmat", vertices=1 << 24, edges=1 << 28, iterations=50, cus=0),
        dict(name="pagerank_largest", kind="pagerank", graph="rmat", vertices=1 << 26, edges=1 << 30, iterations=100, cus=0),
        # a uniform graph on a quarter of the compute units (the cap a user gives the side stream)
        dict(name="pagerank_uniform_64cu", kind="pagerank", graph="uniform", vertices=1 << 23, edges=1 << 28, iterations=100, cus=64),
        # what InitSideTask costs before the first iteration of a graph
        dict(name="new_graph", kind="new_graph", graph="rmat", vertices=1 << 22, edges=1 << 26, iterations=1, cus=0),
        # a side task from registration to stop, steps planned, gated and timed by the runtime
        dict(name="harvest_task", kind="harvest", graph="rmat", vertices=1 << 18, edges=1 << 22, iterations=30, cus=0),
        # the rating graph of the benchmark's second workload, and a small one with uneven sides
        dict(name="sgd_large", kind="sgd", users=1 << 20, items=1 << 20, edges=1 << 24, factors=64, iterations=1),
        dict(name="sgd_small", kind="sgd", users=20_011, items=5_003, edges=300_000, factors=16, iterations=4),
        # the stage's bursts: four transformer layers, hidden 4096, one sequence of 2048 tokens; and one small product
        dict(name="load_h4096", kind="load", layers=4, hidden=4096, ffn=16384, tokens=2048),
        dict(name="gemm_small", kind="gemm", m=512, n=768, k=1024),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["pagerank", "new_graph", "harvest", "sgd", "load", "gemm"], [10, 2, 2, 5, 2, 3])[0]
    if kind in ("pagerank", "new_graph", "harvest"):
        vertices = _log_uniform(rng, 1 << 12, {"pagerank": 1 << 24, "new_graph": 1 << 23, "harvest": 1 << 21}[kind])
        edges = min(int(vertices * math.exp(rng.uniform(math.log(4), math.log(40)))), 1 << 28)
        return dict(kind=kind, graph=rng.choice(["rmat", "rmat", "uniform"]), vertices=vertices, edges=edges,
                    iterations=rng.randint(1, 4) if kind == "new_graph" else rng.randint(10, 50),
                    cus=rng.choice([0, 0, 0, 64, 128]))
    if kind == "sgd":
        users, items = _log_uniform(rng, 1 << 11, 1 << 20), _log_uniform(rng, 1 << 11, 1 << 20)
        edges = int(min(1 << 24, users * items // 8, math.sqrt(users * items) * math.exp(rng.uniform(math.log(8), math.log(64)))))
        return dict(kind="sgd", users=users, items=items, edges=edges, factors=rng.choice([16, 32, 64, 64]), iterations=rng.randint(1, 3))
    if kind == "load":
        hidden = 256 * rng.randint(4, 24)
        return dict(kind="load", layers=rng.randint(1, 4), hidden=hidden, ffn=hidden * rng.choice([2, 4]), tokens=256 * rng.randint(2, 16))
    return dict(kind="gemm", m=256 * _log_uniform(rng, 1, 32), n=256 * _log_uniform(rng, 1, 64), k=64 * _log_uniform(rng, 1, 256))


# ---- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _scatter_ids(raw, bits, n, gen):
    """Ids of 2**bits values onto 0 .. n - 1 (int64): a random permutation, folded where n is no power of two."""
    return torch.randperm(1 << bits, generator=gen, device="cuda")[raw] % n


def _rmat(n_src, n_dst, edges, gen):
    """Edge chunks (src, dst) of an R-MAT graph; the wider side gets the extra levels."""
    sb, db = (n_src - 1).bit_length(), (n_dst - 1).bit_length()
    for first in range(0, edges, 1 << 26):
        n = min(1 << 26, edges - first)
        src = torch.zeros(n, dtype=torch.int32, device="cuda")
        dst = torch.zeros(n, dtype=torch.int32, device="cuda")
        for level in range(max(sb, db)):
            x = torch.rand(n, generator=gen, device="cuda")
            down = x >= 0.76
            right = ((x >= 0.57) & ~down) | (x >= 0.95)
            if level < sb:
                src.mul_(2).add_(down)
            if level < db:
                dst.mul_(2).add_(right)
        yield src, dst


def _csr(case, seed):
    """In-edge CSR (row_ptr, col, out_degree), sources ascending inside a row, multi-edges kept."""
    n, edges = case["vertices"], case["edges"]
    gen = _gen(seed)
    bits = max(1, (n - 1).bit_length())
    keys = torch.empty(edges, dtype=torch.int64, device="cuda")
    if case["graph"] == "rmat":
        perm = torch.randperm(1 << bits, generator=gen, device="cuda") % n
        at = 0
        for src, dst in _rmat(n, n, edges, gen):
            keys[at:at + len(src)] = perm[dst] << bits
            keys[at:at + len(src)] |= perm[src]
            at += len(src)
    else:
        for first in range(0, edges, 1 << 26):
            e = torch.arange(first, min(edges, first + (1 << 26)), device="cuda")
            keys[first:first + len(e)] = torch.randint(0, n, (len(e),), generator=gen, device="cuda") << bits
            keys[first:first + len(e)] |= e % n
    keys = torch.sort(keys).values
    rows = torch.arange(n + 1, device="cuda") << bits
    row_ptr = torch.searchsorted(keys, rows).to(torch.int32)
    col = torch.empty(edges, dtype=torch.int32, device="cuda")
    for first in range(0, edges, 1 << 26):
        col[first:first + (1 << 26)] = keys[first:first + (1 << 26)] & ((1 << bits) - 1)
    del keys
    by_source = torch.sort(col).values
    ends = torch.searchsorted(by_source, torch.arange(n + 1, dtype=torch.int32, device="cuda"))
    return row_ptr, col, (ends[1:] - ends[:-1]).to(torch.int32)


def _ratings(case, seed):
    """CSR by user (row_ptr, item, rating), items ascending and distinct inside a row, and starting factors."""
    users, items, factors = case["users"], case["items"], case["factors"]
    gen = _gen(seed)
    ub, ib = (users - 1).bit_length(), (items - 1).bit_length()
    up = torch.randperm(1 << ub, generator=gen, device="cuda") % users
    ip = torch.randperm(1 << ib, generator=gen, device="cuda") % items
    keys = torch.unique(torch.cat([(up[s] << 32) | ip[d] for s, d in _rmat(users, items, case["edges"], gen)]))
    u, i = keys >> 32, keys & 0xFFFFFFFF
    row_ptr = torch.searchsorted(u, torch.arange(users + 1, device="cuda")).to(torch.int32)
    a = torch.randn(users, 4, generator=gen, device="cuda") / 2
    b = torch.randn(items, 4, generator=gen, device="cuda") / 2
    rating = 3.0 + (a[u] * b[i]).sum(1) + 0.1 * torch.randn(len(u), generator=gen, device="cuda")
    P = torch.rand(users, factors, generator=gen, device="cuda") / math.sqrt(factors)
    Q = torch.rand(items, factors, generator=gen, device="cuda") / math.sqrt(factors)
    return row_ptr, i.to(torch.int32), rating, P, Q


class State:
    """What the program holds between calls; gives the library's objects back when it is dropped."""

    def __init__(self, case):
        self.case = case
        self.task = self.ctx = self.load = self.stream = None

    def __del__(self):
        if isinstance(self.task, fr.SgdTask):
            self.task.fr_sgd_destroy()
        elif self.task is not None:
            self.task.fr_pagerank_destroy()
        if self.load is not None:
            self.load.fr_load_destroy()
        if self.ctx is not None:
            self.ctx.fr_destroy()


def _pagerank_task(s, max_runs=0):
    return fr.PageRankTask(s.case["vertices"], s.case["edges"], s.row_ptr, s.col, s.out_degree, s.ranks, damping=DAMPING,
                           iterations=s.case["iterations"], max_runs=max_runs)


def prepare(case, seed):
    s = State(case)
    kind = case["kind"]
    if kind in ("pagerank", "new_graph", "harvest"):
        s.row_ptr, s.col, s.out_degree = _csr(case, seed)
        s.ranks = torch.zeros(case["vertices"], dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        torch.cuda.empty_cache()              # the library allocates beside torch
        if case["cus"] or kind == "harvest":
            s.ctx = fr.Context(device_id=0, cu_count=case["cus"], guard_ns=60_000, launch_cost_ns=3_000, time_steps=16, adapt_costs=1,
                               device_gate=1, gate_guard_ns=50_000)
            s.stream = s.ctx.fr_side_stream()
        if kind == "pagerank":
            s.task = _pagerank_task(s)
            s.task.fr_pagerank_run_standalone(0, s.stream)         # builds the layout
    elif kind == "sgd":
        s.row_ptr, s.item, s.rating, s.P, s.Q = _ratings(case, seed)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        s.task = fr.SgdTask(case["users"], case["items"], len(s.item), s.row_ptr, s.item, s.rating, s.P, s.Q, case["factors"],
                            GAMMA, LAMBDA, iterations=case["iterations"])
        s.task.fr_sgd_run_standalone(0)                            # builds the layout
    elif kind == "load":
        shape = dict(layers=case["layers"], hidden=case["hidden"], ffn=case["ffn"], tokens=case["tokens"])
        need = fr.Load.fr_load_workspace_bytes(fr.FR_LOAD_GPT, **shape)
        s.workspace = torch.empty(need // 2, dtype=torch.bfloat16, device="cuda")
        s.load = fr.Load(fr.FR_LOAD_GPT, workspace=s.workspace, seed=seed, **shape)
    else:
        gen = _gen(seed)
        s.A = torch.rand(case["m"], case["k"], generator=gen, device="cuda").mul_(2).sub_(1).to(torch.bfloat16)
        s.B = torch.rand(case["n"], case["k"], generator=gen, device="cuda").mul_(2).sub_(1).to(torch.bfloat16)
        s.C = torch.empty(case["m"], case["n"], dtype=torch.bfloat16, device="cuda")
    return s


# ---- one pass

def _harvest(s):
    task = _pagerank_task(s, max_runs=1)
    tid = s.ctx.fr_task_register(task.ops, task.user, task.profile)
    s.ctx.fr_bubble_begin(fr.fr_now_ns(), 10_000_000_000)
    while s.ctx.fr_query_progress(tid).state == fr.FR_CREATED:
        time.sleep(20e-6)
    s.ctx.fr_bubble_end()
    s.ctx.fr_bubble_begin(fr.fr_now_ns(), 10_000_000_000)
    while True:
        pr = s.ctx.fr_query_progress(tid)
        if pr.runs_completed or pr.state == fr.FR_STOPPED:
            break
        time.sleep(20e-6)
    torch.cuda.ExternalStream(s.stream).synchronize()
    s.ctx.fr_bubble_end()
    s.ctx.fr_task_stop(tid)
    task.fr_pagerank_destroy()
    return s.ranks


def run(s):
    kind = s.case["kind"]
    if kind == "pagerank":
        s.task.fr_pagerank_run_standalone(0, s.stream)
        return s.ranks
    if kind == "new_graph":
        task = _pagerank_task(s)
        task.fr_pagerank_run_standalone(0, s.stream)
        task.fr_pagerank_destroy()
        return s.ranks
    if kind == "harvest":
        return _harvest(s)
    if kind == "sgd":
        s.task.fr_sgd_run_standalone(0)
        return s.P, s.Q
    if kind == "load":
        s.load.fr_load_fp()
        s.load.fr_load_bp()
        return s.workspace
    fr.fr_gemm_bf16(s.A, s.B, s.C, s.A.shape[0], s.B.shape[0], s.A.shape[1])
    return s.C


# ---- what a pass cannot do without

def work(case):
    kind = case["kind"]
    if kind in ("pagerank", "new_graph", "harvest"):
        # an iteration reads the sources and row starts, ranks and out-degrees, and writes the ranks; a new graph's CSR is
        # read once more to be checked
        once = 4 * case["edges"] + 24 * case["vertices"] + 4
        return {"bytes": once * (case["iterations"] + (kind != "pagerank")), "flops": 2 * case["edges"] * case["iterations"]}
    if kind == "sgd":
        # ratings with their items once, both factor matrices read and written once; a dot product and two updates a rating
        once = 8 * case["edges"] + 4 * case["users"] + 8 * case["factors"] * (case["users"] + case["items"])
        return {"bytes": once * case["iterations"], "flops": 10 * case["factors"] * case["edges"] * case["iterations"]}
    if kind == "load":
        T, h, f = case["tokens"], case["hidden"], case["ffn"]
        total = {"bytes": 0, "flops": 0}
        for n, k in ((3 * h, h), (h, h), (f, h), (h, f)):        # forward, data gradient, weight gradient
            total["flops"] += case["layers"] * 3 * 2 * T * n * k
            total["bytes"] += case["layers"] * 3 * 2 * (T * n + T * k + n * k)
        return total
    m, n, k = case["m"], case["n"], case["k"]
    return {"bytes": 2 * (m * k + n * k + m * n), "flops": 2 * m * n * k}


def tolerance(case):
    kind = case["kind"]
    if kind == "sgd":
        return "exact"            # every rounding of an update and the order of updates that share a row are fixed
    if kind in ("load", "gemm"):
        return {"rel": 7e-3, "max": 2e-2}        # outputs rounded to bf16 once (against fp64: 1.7e-3 and 3.9e-3)
    return {"rel": 8e-7, "max": 2e-6}            # fp32 ranks (against fp64: 1.9e-7 and 3.3e-7)
