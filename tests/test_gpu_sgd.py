"""GPU parity of the Graph SGD side task (Section 6.1.4's second graph workload), through the C ABI:
bit for bit against the oracle's fp32 mode (same steps, every rounding fixed), within a tolerance against its fp64
mode, and the same bits however the cells are grouped into launches or harvested in bubbles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2409_06941_amd as fr          # noqa: E402
from oracle import sgd as osgd             # noqa: E402
from workloads import ratings as wl        # noqa: E402

# fp32 against fp64 after a few iterations: every update rounds a handful of times (2^-24 relative each) on factors
# of order 1, a factor row is touched some tens of times per iteration, and the iteration is a contraction for
# these step lengths; measured on the CPU between the oracle's two modes: below 1e-4.
TOL64 = 1e-3


def _dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t.to(dtype) if dtype is not None else t).cuda()


def _task(r, P, Q, F, gamma, lam, K, B, **kw):
    rp, it, ra = _dev(r.row_ptr, torch.int32), _dev(r.item, torch.int32), _dev(r.rating, torch.float32)
    if it.numel() == 0:
        it, ra = torch.zeros(4, dtype=torch.int32, device="cuda"), torch.zeros(4, dtype=torch.float32, device="cuda")
    return fr.SgdTask(r.n_users, r.n_items, r.n_ratings, rp, it, ra, P, Q, F, gamma, lam, iterations=K, blocks=B, **kw)


def _run(r, P0, Q0, F, gamma, lam, K, B, max_cells=0):
    P, Q = _dev(P0), _dev(Q0)
    t = _task(r, P, Q, F, gamma, lam, K, B)
    try:
        t.fr_sgd_run_standalone(0, torch.cuda.current_stream(), max_cells)
        info = t.fr_sgd_info()
    finally:
        t.fr_sgd_destroy()
    return P.cpu().numpy(), Q.cpu().numpy(), info


def _same_bits(a, b):
    return np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32))


@pytest.mark.parametrize("scale,edges,F,B,seed", [(6, 700, 16, 1, 1), (8, 5000, 16, 3, 2), (9, 1 << 14, 32, 8, 3),
                                                   (10, (1 << 16) + 77, 64, 16, 4), (12, 1 << 17, 64, 37, 5)])
def test_factors_match_the_oracle(scale, edges, F, B, seed):
    r = wl.rmat_ratings(scale, edges, seed=seed)
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=seed)
    gamma, lam, K = 0.02, 0.03, 3
    print("case U=I=%d E=%d F=%d B=%d" % (r.n_users, r.n_ratings, F, B), flush=True)
    P, Q, info = _run(r, P0, Q0, F, gamma, lam, K, B)
    assert info.blocks == B
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, gamma, lam, K, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)
    P64, Q64 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, gamma, lam, K, B)
    assert np.abs(P - P64).max() <= TOL64 and np.abs(Q - Q64).max() <= TOL64
    assert osgd.rmse(r.row_ptr, r.item, r.rating, P, Q) < osgd.rmse(r.row_ptr, r.item, r.rating, P0, Q0)


@pytest.mark.parametrize("max_cells", [1, 5, 64])
def test_any_grouping_of_cells_into_launches_gives_identical_bits(max_cells):
    r = wl.rmat_ratings(11, 1 << 16, seed=6)
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, 32, seed=6)
    whole = _run(r, P0, Q0, 32, 0.02, 0.03, 2, 24)
    parts = _run(r, P0, Q0, 32, 0.02, 0.03, 2, 24, max_cells)
    assert _same_bits(whole[0], parts[0]) and _same_bits(whole[1], parts[1])


def test_layout_facts_and_default_blocks():
    r = wl.rmat_ratings(12, 1 << 18, seed=7)
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, 16, seed=7)
    P, Q = _dev(P0), _dev(Q0)
    t = _task(r, P, Q, 16, 0.01, 0.0, 1, 0)
    t.fr_sgd_run_standalone(0, torch.cuda.current_stream())
    info = t.fr_sgd_info()
    B = info.blocks
    assert 1 <= B <= 1024 and r.n_ratings // (B * B) >= 32 and r.n_ratings // (4 * B * B) < 32     # largest power of two that fits
    us, is_ = t.fr_sgd_block_starts(0), t.fr_sgd_block_starts(1)
    ous, ois = osgd.blocks(r.row_ptr, r.item, r.n_items, B)
    assert us == list(ous) and is_ == list(ois)
    users = np.repeat(np.arange(r.n_users), np.diff(r.row_ptr))
    a = np.searchsorted(np.array(us[1:B]), users, side="right")
    b = np.searchsorted(np.array(is_[1:B]), r.item, side="right")
    total, largest = 0, 0
    for s in (0, 1, B - 1):
        sizes = t.fr_sgd_cell_sizes(s)
        want = np.bincount(a[(b - a) % B == s], minlength=B)
        assert sizes == list(want)
    for s in range(B):
        sizes = t.fr_sgd_cell_sizes(s)
        total += sum(sizes); largest = max(largest, max(sizes))
    assert total == r.n_ratings and largest == info.largest_cell
    assert largest < 4 * r.n_ratings / (B * B)                      # blocks of equal numbers of ratings keep the cells close
    assert info.bytes_resident >= 12 * r.n_ratings and info.bytes_peak >= info.bytes_resident
    t.fr_sgd_destroy()


def test_no_ratings_leaves_the_factors_alone():
    r = wl.Ratings(5, 7, 0, np.zeros(6, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    P0, Q0 = wl.initial_factors(5, 7, 16, seed=1)
    P, Q, _ = _run(r, P0, Q0, 16, 0.1, 0.1, 2, 2)
    assert _same_bits(P, P0) and _same_bits(Q, Q0)


# A cell without ratings has no entries: nothing may be read from its LDS, which holds what an earlier workgroup left, or is
# none at all where no cell of the task has ratings (the factors keep their bits either way; what this runs is the path)
@pytest.mark.parametrize("F", [16, 32, 64])
@pytest.mark.parametrize("pairs,B", [([], 4), ([(3, 2)], 4), ([(0, 0), (0, 1), (5, 6)], 7), ([(k, (5 * k) % 40) for k in range(40)], 40)])
def test_cells_without_ratings_are_left_alone(pairs, B, F):
    print("case", len(pairs), B, F, flush=True)
    r = _dense(pairs, 41, 41, seed=3)
    P0, Q0 = wl.initial_factors(41, 41, F, seed=F)
    P, Q, info = _run(r, P0, Q0, F, 0.02, 0.03, 3, B)
    assert info.blocks == B and info.largest_cell <= len(pairs) < B * B      # most cells have none
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 3, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


def test_malformed_ratings_are_refused():
    r = wl.rmat_ratings(6, 500, seed=8)
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, 16, seed=1)
    with pytest.raises(fr.FreeRideError):
        _task(r, _dev(P0), _dev(Q0), 8, 0.1, 0.1, 1, 1)                        # unsupported number of factors
    u = int(np.argmax(np.diff(r.row_ptr) >= 2))
    swapped = r.item.copy()
    e = r.row_ptr[u]
    swapped[e], swapped[e + 1] = swapped[e + 1], swapped[e]                     # a row whose items do not ascend
    for bad_items in (swapped, np.where(np.arange(r.n_ratings) == 3, r.n_items, r.item).astype(np.int32)):
        bad = wl.Ratings(r.n_users, r.n_items, r.n_ratings, r.row_ptr, bad_items, r.rating)
        P, Q = _dev(P0), _dev(Q0)
        t = _task(bad, P, Q, 16, 0.1, 0.1, 1, 2)
        with pytest.raises(fr.FreeRideError) as ei:
            t.fr_sgd_run_standalone(0, torch.cuda.current_stream())
        assert ei.value.code == fr.FR_ERR_ARG
        t.fr_sgd_destroy()
        assert _same_bits(P.cpu().numpy(), P0)                                 # nothing ran


def test_harvested_in_bubbles_gives_the_standalone_bits():
    from workloads import configs
    cfg = configs.by_name("cfg1")
    r = wl.rmat_ratings(12, 1 << 17, seed=9)
    F, gamma, lam, K, B, runs = 32, 0.02, 0.03, 2, 16, 2
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=9)
    # reference: `runs` standalone runs in a row (the factors carry over)
    Pr, Qr = _dev(P0), _dev(Q0)
    t_ref = _task(r, Pr, Qr, F, gamma, lam, K, B)
    ns = [t_ref.fr_sgd_run_standalone(0, torch.cuda.current_stream(), want_ns=True) for _ in range(runs)]
    info = t_ref.fr_sgd_info()
    sizes = [t_ref.fr_sgd_cell_sizes(s) for s in range(B)]
    assert info.chain_ratings == sum(max(row) for row in sizes)
    t_ref.fr_sgd_destroy()
    # cost model from the measured run: the cells of a stratum run side by side, so a step of any number of them takes
    # about a stratum's time (the floor), and a whole stratum's cells add up to the same
    stratum_ns = min(ns) / (K * B)
    fs_per_rating = int(0.5 * stratum_ns * 1e6 / (r.n_ratings / B))
    fs_chain = int(1.5 * min(ns) * 1e6 / info.chain_ratings)                 # a step takes as long as its largest cell
    floor_ns = int(0.75 * stratum_ns) + 10_000
    print("stratum %.1f us, %.2f us per rating of a cell" % (stratum_ns / 1e3, stratum_ns / 1e3 / (r.n_ratings / B / B)), flush=True)

    P, Q = _dev(P0), _dev(Q0)
    ctx = fr.Context(device_id=0, guard_ns=200_000, launch_cost_ns=20_000, max_chunk_ns=0, time_steps=1,
                     mem_available_bytes=1 << 40)
    task = _task(r, P, Q, F, gamma, lam, K, B, max_runs=runs, mem_limit_bytes=1 << 30, fs_per_rating=fs_per_rating,
                 min_step_ns=floor_ns, fs_per_chain_rating=fs_chain)
    tid = ctx.fr_task_register(task.ops, task.user, task.profile)
    import time
    ctx.fr_bubble_begin(fr.fr_now_ns(), 2_000_000_000)
    t_end = time.time() + 30
    while ctx.fr_query_progress(tid).state == fr.FR_CREATED and time.time() < t_end:
        time.sleep(0.001)
    ctx.fr_bubble_end()
    assert ctx.fr_query_progress(tid).state == fr.FR_PAUSED
    stream = torch.cuda.Stream()
    load = fr.Load(fr.FR_LOAD_BUSYWAIT, fp_ns=cfg.busy_fp_ns, bp_ns=cfg.busy_bp_ns)
    stage = fr.Stage(fr.FR_SCHED_1F1B, cfg.p, cfg.m, cfg.stage, cfg.busy_fp_ns, cfg.busy_bp_ns, load, stream)
    overruns = 0
    for ep in range(40):
        print("epoch", ep, flush=True)
        overruns += stage.fr_stage_run_epoch(ctx).overruns
        if ctx.fr_query_progress(tid).runs_completed >= runs:
            break
    time.sleep(0.05)
    pr = ctx.fr_query_progress(tid)
    log = ctx.fr_event_log()
    ctx.fr_task_stop(tid)
    got_P, got_Q = P.cpu().numpy(), Q.cpu().numpy()
    task.fr_sgd_destroy(); stage.fr_stage_destroy(); load.fr_load_destroy(); ctx.fr_destroy()
    assert pr.runs_completed == runs and overruns == 0 and pr.deadline_misses == 0
    chunks = [e for e in log if e.kind == fr.FR_EV_CHUNK]
    assert sum(e.work_units for e in chunks) == runs * K * r.n_ratings == pr.work_units_done
    assert len(chunks) >= runs * K * B                         # a step never spans two strata
    ceil_ns = lambda fs: max(1, -(-fs // 10**6))
    for e in chunks:                                           # the documented cost rule, on every step of the log
        row = sizes[e.segment % B][e.tile0:e.tile1]
        want = max(sum(ceil_ns(n * fs_per_rating) for n in row), floor_ns, ceil_ns(max(row) * fs_chain))
        assert e.modelled_ns == want + 20_000 and e.work_units == sum(row)
    assert _same_bits(got_P, Pr.cpu().numpy()) and _same_bits(got_Q, Qr.cpu().numpy())


@pytest.mark.timeout(600)
def test_full_size_of_the_benchmark_gives_the_oracles_bits():
    # the workload of `bench.py --side-task sgd` (2^20 x 2^20, 16.1 M ratings, 64 factors, blocks chosen by the library),
    # one iteration, every factor compared bit for bit with the oracle's fp32 mode (about half a minute of CPU)
    r = wl.rmat_ratings(20, 1 << 24, seed=1)
    F, gamma, lam = 64, 0.01, 0.02
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=1)
    print("case U=I=%d E=%d F=%d" % (r.n_users, r.n_ratings, F), flush=True)
    P, Q, info = _run(r, P0, Q0, F, gamma, lam, 1, 0)
    assert info.blocks == 512
    print("gpu done, oracle running", flush=True)
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, gamma, lam, 1, info.blocks, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)
    assert not _same_bits(P, P0)


def test_pagerank_and_sgd_queued_on_one_worker_run_one_after_the_other():
    # Algorithms 1 and 2 with two different side tasks: both are accepted, the first one submitted runs until it reports
    # that it has finished, then the second takes the bubbles; each ends with the bits of its standalone run.
    import time
    from oracle.pagerank import pagerank
    from workloads import configs, graphs
    cfg = configs.by_name("cfg1")
    g = graphs.rmat_csr(13, 1 << 17, seed=3)
    r = wl.rmat_ratings(11, 1 << 16, seed=10)
    F, gamma, lam, K_sgd, B, K_pr = 16, 0.02, 0.03, 2, 8, 10
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=10)
    Pr, Qr, _ = _run(r, P0, Q0, F, gamma, lam, K_sgd, B)                        # SGD reference bits
    rp, col, od = _dev(g.row_ptr, torch.int32), _dev(g.col, torch.int32), _dev(g.out_degree, torch.int32)
    ranks = torch.zeros(g.n_vertices, dtype=torch.float32, device="cuda")
    P, Q = _dev(P0), _dev(Q0)
    ctx = fr.Context(device_id=0, guard_ns=200_000, launch_cost_ns=20_000, max_chunk_ns=0, time_steps=1, mem_available_bytes=1 << 40)
    pr_task = fr.PageRankTask(g.n_vertices, g.n_edges, rp, col, od, ranks, iterations=K_pr, max_runs=1, mem_limit_bytes=1 << 30,
                              fs_per_edge=400_000, fs_per_message=400_000, fs_per_vertex=300_000, finish_tile_ns=15000)
    sgd_task = _task(r, P, Q, F, gamma, lam, K_sgd, B, max_runs=1, mem_limit_bytes=1 << 30, fs_per_rating=100_000_000, min_step_ns=200_000)
    t_pr = ctx.fr_task_register(pr_task.ops, pr_task.user, pr_task.profile)
    t_sgd = ctx.fr_task_register(sgd_task.ops, sgd_task.user, sgd_task.profile)
    assert ctx.fr_query_progress(t_pr).state == fr.FR_CREATED and ctx.fr_query_progress(t_sgd).state == fr.FR_SUBMITTED
    stream = torch.cuda.Stream()
    load = fr.Load(fr.FR_LOAD_BUSYWAIT, fp_ns=cfg.busy_fp_ns, bp_ns=cfg.busy_bp_ns)
    stage = fr.Stage(fr.FR_SCHED_1F1B, cfg.p, cfg.m, cfg.stage, cfg.busy_fp_ns, cfg.busy_bp_ns, load, stream)
    order = []
    for ep in range(30):
        print("epoch", ep, flush=True)
        stage.fr_stage_run_epoch(ctx)
        a, b = ctx.fr_query_progress(t_pr), ctx.fr_query_progress(t_sgd)
        if a.runs_completed and "pagerank" not in order:
            order.append("pagerank")
            assert b.runs_completed == 0                                       # the second task has not finished before the first
        if b.runs_completed:
            order.append("sgd")
            break
    time.sleep(0.05)
    a, b = ctx.fr_query_progress(t_pr), ctx.fr_query_progress(t_sgd)
    if b.state != fr.FR_STOPPED:
        ctx.fr_task_stop(t_sgd)
    if a.state != fr.FR_STOPPED:
        ctx.fr_task_stop(t_pr)
    got_ranks, got_P, got_Q = ranks.cpu().numpy(), P.cpu().numpy(), Q.cpu().numpy()
    pr_task.fr_pagerank_destroy(); sgd_task.fr_sgd_destroy(); stage.fr_stage_destroy(); load.fr_load_destroy(); ctx.fr_destroy()
    assert order == ["pagerank", "sgd"] and a.runs_completed == 1 and b.runs_completed == 1
    assert a.state == fr.FR_STOPPED and a.last_error == fr.FR_OK                # finished and gave way to the next in the queue
    assert a.overruns == 0 and b.overruns == 0
    assert np.abs(got_ranks.astype(np.float64) - pagerank(g.row_ptr, g.col, g.out_degree, 0.85, K_pr)).max() <= 1e-5
    assert _same_bits(got_P, Pr) and _same_bits(got_Q, Qr)


def test_device_gate_refuses_late_sgd_steps_and_the_factors_keep_their_bits():
    # The model claims a quarter of what the strata take, so the host keeps enqueueing steps that cannot end inside the
    # bubble; with the device gate the late ones do nothing and the task is rewound to the first of them.  SGD updates
    # its factors in place, so a step that ran twice, or half, would show in the bits.
    import time
    r = wl.rmat_ratings(12, 1 << 17, seed=11)
    F, gamma, lam, K, B = 32, 0.02, 0.03, 2, 16
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=11)
    Pr, Qr = _dev(P0), _dev(Q0)
    t_ref = _task(r, Pr, Qr, F, gamma, lam, K, B)
    t_ref.fr_sgd_run_standalone(0, torch.cuda.current_stream())
    ns = t_ref.fr_sgd_run_standalone(0, torch.cuda.current_stream(), want_ns=True)
    t_ref.fr_sgd_destroy()
    Pr, Qr, _ = _run(r, P0, Q0, F, gamma, lam, K, B)                            # one run from the start: the reference bits
    stratum_ns = ns / (K * B)
    low = 0.25
    P, Q = _dev(P0), _dev(Q0)
    ctx = fr.Context(device_id=0, guard_ns=20_000, launch_cost_ns=5_000, max_chunk_ns=0, time_steps=4, device_gate=1,
                     mem_available_bytes=1 << 40)
    task = _task(r, P, Q, F, gamma, lam, K, B, max_runs=1, mem_limit_bytes=1 << 30,
                 fs_per_rating=int(low * stratum_ns * 1e6 / (r.n_ratings / B)), min_step_ns=int(low * stratum_ns))
    tid = ctx.fr_task_register(task.ops, task.user, task.profile)
    ctx.fr_bubble_begin(fr.fr_now_ns(), 2_000_000_000)
    t_end = time.time() + 30
    while ctx.fr_query_progress(tid).state == fr.FR_CREATED and time.time() < t_end:
        time.sleep(0.001)
    ctx.fr_bubble_end()
    stream = torch.cuda.Stream()
    f_ns, b_ns = 1_000_000, 2_000_000
    load = fr.Load(fr.FR_LOAD_BUSYWAIT, fp_ns=f_ns, bp_ns=b_ns)
    stage = fr.Stage(fr.FR_SCHED_1F1B, 4, 8, 2, f_ns, b_ns, load, stream)
    for ep in range(40):
        print("epoch", ep, flush=True)
        stage.fr_stage_run_epoch(ctx)
        time.sleep(0.01)
        if ctx.fr_query_progress(tid).runs_completed >= 1:
            break
    time.sleep(0.05)
    pr = ctx.fr_query_progress(tid)
    log = ctx.fr_event_log()
    if pr.state != fr.FR_STOPPED:
        ctx.fr_task_stop(tid)
    got_P, got_Q = P.cpu().numpy(), Q.cpu().numpy()
    task.fr_sgd_destroy(); stage.fr_stage_destroy(); load.fr_load_destroy(); ctx.fr_destroy()
    chunks = [e for e in log if e.kind == fr.FR_EV_CHUNK]
    refused = [e for e in log if e.kind == fr.FR_EV_REFUSED]
    print("steps", pr.steps, "refused", pr.steps_refused, "runs", pr.runs_completed, flush=True)
    assert pr.runs_completed == 1 and pr.steps_refused > 0 and len(refused) == pr.steps_refused
    assert pr.work_units_done == sum(e.work_units for e in chunks) - sum(e.work_units for e in refused) == K * r.n_ratings
    assert _same_bits(got_P, Pr) and _same_bits(got_Q, Qr)
    # and against the oracle itself, not only against another GPU run: the bits of its fp32 mode, the values of its fp64 mode
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, gamma, lam, K, B, ordered_fp32=True)
    assert _same_bits(got_P, P32) and _same_bits(got_Q, Q32)
    P64, Q64 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, gamma, lam, K, B)
    assert np.abs(got_P - P64).max() <= TOL64 and np.abs(got_Q - Q64).max() <= TOL64


def _dense(pairs, n_users, n_items, seed):
    pairs = sorted(set(pairs))
    row_ptr = np.zeros(n_users + 1, np.int64)
    np.add.at(row_ptr, np.array([u for u, _ in pairs], np.int64) + 1, 1)
    rating = np.random.default_rng(seed).uniform(1, 5, len(pairs)).astype(np.float32)
    return wl.Ratings(n_users, n_items, len(pairs), np.cumsum(row_ptr).astype(np.int32), np.array([i for _, i in pairs], np.int32), rating)


def _limits(r, F, B, seed=4):
    """What the task's own buffers come to beside the caller's, under a limit: (resident, peak), and the factors."""
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=seed)
    caller = 4 * (r.n_users + 1) + 8 * r.n_ratings + 4 * F * (r.n_users + r.n_items)

    def run(own_limit):
        P, Q = _dev(P0), _dev(Q0)
        t = _task(r, P, Q, F, 0.02, 0.03, 2, B, mem_limit_bytes=caller + own_limit)
        try:
            t.fr_sgd_run_standalone(0, torch.cuda.current_stream())
            info = t.fr_sgd_info()
        finally:
            t.fr_sgd_destroy()
        return info.bytes_resident - caller, info.bytes_peak - caller, P.cpu().numpy(), Q.cpu().numpy()
    return run


@pytest.mark.parametrize("F,B", [(16, 64), (64, 64), (32, 40)])
def test_a_limit_without_room_for_the_rounds_takes_the_small_layout(F, B):
    # 20 bytes a rating for the sort (and its scratch) and 4 per cell are what the ratings in a row need, 12 of them for good
    r = wl.rmat_ratings(13, 300_000, seed=12)
    run = _limits(r, F, B)
    resident, peak, P, Q = run(1 << 40)
    assert resident > 16 * r.n_ratings                            # rounds
    enough = 32 * r.n_ratings + 4 * B * B + (1 << 17)
    assert peak > enough                                          # (else this test looks at nothing)
    for limit in (enough, peak - 1):
        print("case", F, B, limit, flush=True)
        small, small_peak, P2, Q2 = run(limit)
        assert small <= 12 * r.n_ratings + 4 * B * B + 8 * B + 4096 and small_peak <= limit
        assert _same_bits(P, P2) and _same_bits(Q, Q2)
    with pytest.raises(fr.FreeRideError) as e:
        run(19 * r.n_ratings)
    assert e.value.code == fr.FR_ERR_OOM


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("F", [16, 64])
def test_sparse_cells_stay_small(F, dense):
    B, n = 256, 1 << 13
    rng = np.random.default_rng(5)
    if dense:
        # 128 ratings a block: the first 128 users and items, a diagonal, are cell (0, 0) with 256 rows, the longest record
        # there is; the others are spread over the other cells, half of which have none
        pairs = {(k, k) for k in range(128)}
        while len(pairs) < 128 * B:
            pairs |= set(zip(rng.integers(128, n, 2000).tolist(), rng.integers(128, n, 2000).tolist()))
        r = _dense(sorted(pairs)[:128 * B], n, n, seed=9)
    else:
        r = wl.rmat_ratings(14, 240_000, seed=14)                 # about three a cell
    print("case", F, r.n_ratings, flush=True)
    resident, _, P, Q = _limits(r, F, B)(1 << 40)
    assert resident <= 128 * r.n_ratings + (1 << 16)
    P0, Q0 = wl.initial_factors(r.n_users, r.n_items, F, seed=4)
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 2, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


# where the layout in rounds can go wrong: a batch of one rating, full batches and one more (128, 129), one chain (a single
# user or item), no chain at all (a diagonal: 256 rows and the most LDS), a grid, cells without ratings, and both sides of
# the mean cell size (256) from which on the ratings are worked on one after the other
@pytest.mark.parametrize("F", [16, 32, 64])
@pytest.mark.parametrize("shape,B", [((1, 1), 1), ((1, 128), 1), ((1, 129), 1), ((129, 1), 1), ("diagonal", 1), ((16, 16), 1), ((1, 257), 1),
                                     ((33, 31), 2), ((9, 7), 7)])
def test_rounds_of_a_batch_match_the_oracle(shape, B, F):
    print("case", shape, B, F, flush=True)
    pairs = [(k, k) for k in range(128)] if shape == "diagonal" else [(u, i) for u in range(shape[0]) for i in range(shape[1])]
    n_users, n_items = max(u for u, _ in pairs) + 3, max(i for _, i in pairs) + 2
    r = _dense(pairs, n_users, n_items, seed=len(pairs))
    P0, Q0 = wl.initial_factors(n_users, n_items, F, seed=F)
    P, Q, _ = _run(r, P0, Q0, F, 0.02, 0.03, 3, B)
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 3, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


# rounds one after the other in pieces without a branch (of twelve, six with 32 factors, and of three behind them): chains of as
# many ratings as there are rounds, on both sides of the pieces' ends
@pytest.mark.parametrize("F", [16, 32, 64])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 11, 12, 13, 14, 17, 18, 23, 24, 25, 26, 127])
def test_chains_of_any_length_match_the_oracle(n, F):
    r = _dense([(0, i) for i in range(n)], 1, n, seed=n)
    P0, Q0 = wl.initial_factors(1, n, F, seed=F)
    P, Q, _ = _run(r, P0, Q0, F, 0.02, 0.03, 3, 1)
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 3, 1, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


# from 128 blocks on the next stratum's programs are read ahead: the last stratum reads those of the first, cells without ratings
# and of several batches among them; also on the other side of the line, and cell by cell
@pytest.mark.parametrize("B,F,cells", [(127, 16, 0), (128, 16, 0), (128, 64, 50), (130, 32, 0)])
def test_programs_read_ahead_leave_the_factors_alone(B, F, cells):
    rng = np.random.default_rng(B)
    n = 4000
    pairs = set(zip(rng.integers(0, n, 150_000).tolist(), rng.integers(0, n, 150_000).tolist()))
    pairs |= {(u, i) for u in range(30) for i in range(300)}                     # (cells of more than 128 ratings)
    r = _dense(sorted(pairs), n, n, seed=B)
    P0, Q0 = wl.initial_factors(n, n, F, seed=F)
    print("case", B, F, cells, r.n_ratings, flush=True)
    P, Q, info = _run(r, P0, Q0, F, 0.02, 0.03, 2, B, cells)
    assert info.blocks == B
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 2, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


# from 128 blocks and 16 ratings a cell on the next stratum's programs are read ahead: the last stratum reads those of the first,
# cells without ratings and of several batches among them; also on the other side of the lines (127 blocks, launches of 30 cells)
@pytest.mark.parametrize("B,F,cells", [(127, 16, 0), (128, 16, 0), (128, 64, 50), (128, 64, 30), (130, 32, 0)])
def test_programs_of_large_cells_read_ahead_leave_the_factors_alone(B, F, cells):
    rng = np.random.default_rng(B)
    n = 4000
    pairs = set(zip(rng.integers(0, n, 290_000).tolist(), rng.integers(0, n, 290_000).tolist()))
    pairs |= {(u, i) for u in range(30) for i in range(300)}                     # (cells of more than 128 ratings)
    r = _dense(sorted(pairs), n, n, seed=B)
    P0, Q0 = wl.initial_factors(n, n, F, seed=F)
    print("case", B, F, cells, r.n_ratings, flush=True)
    P, Q, info = _run(r, P0, Q0, F, 0.02, 0.03, 2, B, cells)
    assert info.blocks == B and r.n_ratings >= 16 * B * B
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 2, B, ordered_fp32=True)
    assert _same_bits(P, P32) and _same_bits(Q, Q32)


# 16 factors: up to seven cells a unit in a launch take one kernel, eight another
@pytest.mark.parametrize("B,cells", [(56, 0), (57, 0), (64, 0), (64, 57), (64, 56)])
def test_many_cells_on_few_units_match_the_oracle(B, cells):
    rng = np.random.default_rng(B)
    n = 900
    pairs = set(zip(rng.integers(0, n, 90_000).tolist(), rng.integers(0, n, 90_000).tolist()))
    pairs |= {(u, i) for u in range(20) for i in range(200)}                     # (cells of more than 128 ratings)
    r = _dense(sorted(pairs), n, n, seed=B)
    P0, Q0 = wl.initial_factors(n, n, 16, seed=3)
    P, Q = _dev(P0), _dev(Q0)
    print("case", B, cells, r.n_ratings, flush=True)
    ctx = fr.Context(device_id=0, cu_count=8)
    t = _task(r, P, Q, 16, 0.02, 0.03, 3, B)
    try:
        t.fr_sgd_run_standalone(0, ctx.fr_side_stream(), cells)
        assert t.fr_sgd_info().blocks == B
    finally:
        t.fr_sgd_destroy()
        ctx.fr_destroy()
    P32, Q32 = osgd.sgd(r.row_ptr, r.item, r.rating, P0, Q0, 0.02, 0.03, 3, B, ordered_fp32=True)
    assert _same_bits(P.cpu().numpy(), P32) and _same_bits(Q.cpu().numpy(), Q32)
