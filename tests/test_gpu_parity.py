"""Parity of the HIP path (through the C ABI) with the CPU oracle.

Bars: validity masks, memory bytes and the selected plans are bit-exact; iteration
time and cost agree within a relative 1e-5 (fp32 on the device, fp64 in the oracle).
The constraint bit is decided in floating point, so candidates whose constrained
value lies within 1e-5 of the bound are exempt from the bit-5 comparison.
"""
import os

import numpy as np
import pytest

from oracle.oracle import MAX_THROUGHPUT, MIN_COST, Oracle
from paper_2504_17096_amd import workloads as W
from tests.helpers import make_problem, wide_problem

pytestmark = pytest.mark.gpu

REL = 1e-5
THREADS = min(16, os.cpu_count() or 1)


def _plan(prob):
    from paper_2504_17096_amd.binding import Plan
    return Plan(prob)


def gpu_eval(torch, plan, first, count, indices=None, objective=MAX_THROUGHPUT, bound=None):
    dev = "cuda:0"
    t = torch.empty(count, dtype=torch.float32, device=dev)
    c = torch.empty(count, dtype=torch.float32, device=dev)
    m = torch.empty(count, dtype=torch.int64, device=dev)
    k = torch.empty(count, dtype=torch.int32, device=dev)
    d_idx = None
    if indices is not None:
        d_idx = torch.from_numpy(np.asarray(indices, dtype=np.uint64).view(np.int64)).to(dev)
    stream = torch.cuda.current_stream().cuda_stream
    plan.eval_batch(first, count, d_indices=d_idx, objective=objective, bound=bound,
                    d_time=t, d_cost=c, d_mem=m, d_mask=k, stream=stream)
    torch.cuda.synchronize()
    return (t.cpu().numpy(), c.cpu().numpy(), m.cpu().numpy().view(np.uint64),
            k.cpu().numpy().view(np.uint32))


def assert_eval_parity(got, want, objective=MAX_THROUGHPUT, bound=None):
    gt, gc, gm, gk = got
    wt, wc, wm, wk = want
    hard = np.uint32(0xF)
    assert np.array_equal(gk & hard, wk & hard), "integer-decided mask bits differ"
    assert np.array_equal(gm, wm), "memory bytes differ"
    fin = np.isfinite(wt)
    assert np.array_equal(np.isfinite(gt), fin) and np.array_equal(np.isfinite(gc), fin)
    assert np.all(np.abs(gt[fin] - wt[fin]) <= REL * wt[fin])
    assert np.all(np.abs(gc[fin] - wc[fin]) <= REL * wc[fin])
    if bound is None:
        assert np.array_equal(gk, wk)
    else:
        val = wc if objective == MAX_THROUGHPUT else 1.0 / wt
        care = fin & (np.abs(val - bound) > REL * bound)
        assert np.array_equal(gk[care] & 32, wk[care] & 32)
        if np.count_nonzero(fin) >= 5000:  # the exempt band must stay thin
            assert np.count_nonzero(fin & ~care) < 0.01 * np.count_nonzero(fin)
    return float(np.max(np.abs(gt[fin] - wt[fin]) / wt[fin], initial=0.0))


def check_result(res, want, orc):
    """A sailor_result against the oracle's evaluation and decoding of the same index."""
    assert res.index == want.index
    assert res.mask == 0 and res.peak_mem_bytes == want.peak_mem
    assert res.iter_time_s == pytest.approx(want.iter_time, rel=1e-9)
    assert res.cost_per_iter == pytest.approx(want.cost, rel=1e-9)
    cfg = orc.decode(want.index)
    assert (res.pp, res.tp, res.dp, res.mb) == (cfg.pp, cfg.tp, cfg.dp, cfg.mb)
    assert (res.pp_index, res.tp_index, res.dp_index, res.mb_index) == (
        cfg.pp_idx, cfg.tp_idx, cfg.dp_idx, cfg.mb_idx)
    assert (res.partition, res.n_segments, res.cut, res.pool) == (
        cfg.partition, cfg.n_segments, cfg.cut, cfg.pool)
    assert (res.seg_tp, res.seg_tp_index) == (cfg.seg_tp, cfg.seg_tp_idx)
    # zone and the two replica types of every segment, from the documented pool numbering
    import itertools
    G = orc._prob.n_types
    xt = [(a, a) for a in range(G)] + (list(itertools.combinations(range(G), 2))
                                        if getattr(orc._prob, "mixed_types", False) else [])
    for j in range(3):
        if cfg.pool[j] < 0:
            assert (res.zone[j], res.type_a[j], res.type_b[j]) == (-1, -1, -1)
        else:
            z, (a, b) = cfg.pool[j] // len(xt), xt[cfg.pool[j] % len(xt)]
            assert (res.zone[j], res.type_a[j], res.type_b[j]) == (z, a, b)


def off_data(bound):
    """A bound taken from the data (a median, a quantile) can coincide with one candidate's
    value to the last bit, and `value > bound` at exact equality depends on the order of the
    fp64 additions: move it a hair off."""
    return bound * (1.0 + 1e-7)


def check_topk(got, want, objective, orc=None, bound=None):
    """Same plans in the same order.  Keys that agree to 1e-12 count as ties (the two sides
    add the per-layer times in different orders): tied neighbours may swap, and which of
    the plans tied with the k-th key make the list may differ.  With the oracle at hand,
    every plan the device returns in place of a tied one is re-checked against it."""
    assert len(got) == len(want)
    if not want:
        return
    key = (lambda e: e.iter_time) if objective == MAX_THROUGHPUT else (lambda e: e.cost)
    gkey = (lambda r: r.iter_time_s) if objective == MAX_THROUGHPUT else (lambda r: r.cost_per_iter)
    kth = key(want[-1])
    below = kth * (1.0 - 1e-12)
    assert sorted(r.index for r in got if gkey(r) < below) == sorted(
        e.index for e in want if key(e) < below)
    wanted = {e.index for e in want}
    for r in got:
        if r.index not in wanted:  # stands in for a plan tied with the k-th
            assert orc is not None, "the returned sets differ"
            e = orc.eval_one(r.index, objective=objective, bound=bound)
            assert e.mask == 0 and r.mask == 0
            assert gkey(r) == pytest.approx(key(e), rel=1e-9)
            assert key(e) == pytest.approx(kth, rel=1e-12)
    for r, e in zip(got, want):
        if r.index != e.index:
            assert gkey(r) == pytest.approx(key(e), rel=1e-12)


# ------------------------------------------------------------------ small spaces, exhaustively

PROBLEMS = {
    "cfg1": W.config1,
    "cfg2": W.config2,
    "tiny1": lambda: W.tiny_problem(1),
    "tiny2": lambda: W.tiny_problem(2, n_zones=3),
    "tiny3": lambda: W.tiny_problem(3, uniform_layers=True),
    "tiny4": lambda: W.tiny_problem(4, n_layers=8, n_types=3, seg3_max_pp=8),
    "tiny5": lambda: W.tiny_problem(5, n_layers=12, max_segments=2, with_egress=False),
    "tiny6": lambda: W.tiny_problem(6, n_zones=1, n_types=1),
    "onepool": lambda: make_problem(n_layers=4, max_segments=3, seg3_max_pp=4),
    "wide": wide_problem,
    # every segment with its own TP digit
    "cfg1_segtp": lambda: W.config1().with_per_segment_tp(),
    "cfg2_segtp": lambda: W.config2().with_per_segment_tp(),
    "tiny1_segtp": lambda: W.tiny_problem(1).with_per_segment_tp(),
    "tiny2_segtp": lambda: W.tiny_problem(2, n_zones=3).with_per_segment_tp(),
    "tiny4_segtp": lambda: W.tiny_problem(4, n_layers=8, n_types=3, seg3_max_pp=8).with_per_segment_tp(),
    "onepool_segtp": lambda: make_problem(n_layers=4, max_segments=3, seg3_max_pp=4).with_per_segment_tp(),
    # message-size dependent link bandwidth
    "cfg2_bwpoly": lambda: _with_profile(W.config2()),
    "tiny2_bwpoly": lambda: _with_profile(W.tiny_problem(2, n_zones=3)),
    "tiny4_segtp_bwpoly": lambda: _with_profile(
        W.tiny_problem(4, n_layers=8, n_types=3, seg3_max_pp=8).with_per_segment_tp()),
    # replicas of a stage split over two GPU types
    "cfg2_mixed": lambda: W.config2().with_mixed_types(),
    "tiny1_mixed": lambda: W.tiny_problem(1).with_mixed_types(),
    "tiny4_mixed": lambda: W.tiny_problem(4, n_layers=8, n_types=3, seg3_max_pp=8).with_mixed_types(),
    "tiny2_mixed_segtp_bwpoly": lambda: _with_profile(
        W.tiny_problem(2, n_zones=3).with_mixed_types().with_per_segment_tp()),
    "scarce_mixed": lambda: _scarce(W.tiny_problem(8, n_types=3, n_zones=2).with_mixed_types()),
    # the deepest pipeline the library accepts: 256 stages of one layer each
    "deep256": lambda: _deep(),
}


def _deep():
    rng = np.random.default_rng(256)
    L = 256
    return make_problem(n_layers=L, n_types=2, n_zones=2, mb_list=(1, 2), tp_list=(1, 2), dp_list=(1, 2, 4),
                        pp_list=[64, 255, 256], global_batch=64, max_segments=2, uniform_layers=False,
                        partitions={255: [[2] + [1] * 254, [1] * 127 + [2] + [1] * 127]},
                        t_fwd=rng.uniform(0.5e-3, 2e-3, (2, 2, 2, L)), t_bwd=rng.uniform(1e-3, 4e-3, (2, 2, 2, L)),
                        t_upd=rng.uniform(1e-5, 3e-5, (2, 2, L)),
                        layer_params=rng.integers(1_000_000, 3_000_000, L).astype(np.uint64),
                        act=rng.integers(1_000_000, 9_000_000, (2, 2)).astype(np.uint64), p2p=2_000_000,
                        cap=np.array([2, 1], np.uint64) * np.uint64(1 << 30), avail=np.array([[600, 300], [400, 500]]),
                        bw=np.array([[1e10, 1e9], [2e9, 1e10]]), egress=np.array([[0, 2e-11], [3e-11, 0]]),
                        price=np.array([3.0, 1.5]))


def _scarce(prob):
    """Few GPUs everywhere, so that segments compete for the real pools they share."""
    return prob.with_avail(np.random.default_rng(8).integers(1, 12, prob.avail.shape))


def _with_profile(prob, seed=6):
    return prob.with_bw_poly(W.bandwidth_poly(prob, seed))


@pytest.fixture(scope="module", params=sorted(PROBLEMS))
def case(request, torch_cuda):
    prob = PROBLEMS[request.param]()
    plan = _plan(prob)
    orc = Oracle(prob)
    yield prob, plan, orc
    plan.destroy()


def test_space_size_and_decode(case):
    prob, plan, orc = case
    n = plan.num_candidates()
    assert n == orc.num_candidates
    rng = np.random.default_rng(0)
    for c in [0, n - 1] + rng.integers(0, n, 300).tolist():
        r, cfg = plan.decode(int(c)), orc.decode(int(c))
        assert (r.pp, r.tp, r.dp, r.mb, r.partition, r.n_segments, r.cut, r.pool) == (
            cfg.pp, cfg.tp, cfg.dp, cfg.mb, cfg.partition, cfg.n_segments, cfg.cut, cfg.pool)
        assert (r.seg_tp, r.seg_tp_index) == (cfg.seg_tp, cfg.seg_tp_idx)
    from paper_2504_17096_amd.binding import SAILOR_ERANGE, SailorError
    with pytest.raises(SailorError) as ei:
        plan.decode(n)
    assert ei.value.status == SAILOR_ERANGE


@pytest.mark.parametrize("objective", [MAX_THROUGHPUT, MIN_COST])
def test_eval_batch_whole_space(case, torch_cuda, objective):
    prob, plan, orc = case
    n = orc.num_candidates
    want = orc.eval_batch(objective=objective, n_threads=THREADS)
    got = gpu_eval(torch_cuda, plan, 0, n, objective=objective)
    assert_eval_parity(got, want)
    ok = want[3] == 0
    if ok.any():
        val = want[1] if objective == MAX_THROUGHPUT else 1.0 / want[0]
        bound = off_data(float(np.median(val[ok])))
        want_b = orc.eval_batch(objective=objective, bound=bound, n_threads=THREADS)
        got_b = gpu_eval(torch_cuda, plan, 0, n, objective=objective, bound=bound)
        assert_eval_parity(got_b, want_b, objective, bound)


def test_eval_batch_in_pieces_returns_the_same_bits(case, torch_cuda):
    # a range is cut into units at fixed places of the index space and clipped where it begins
    # and ends inside one: however a range is cut into pieces, the pieces hold the bits of the whole
    prob, plan, orc = case
    n = orc.num_candidates
    rng = np.random.default_rng(11)
    ok = orc.eval_batch()[3] == 0
    bound = None
    if ok.any():
        bound = off_data(float(np.median(orc.eval_batch()[1][ok])))
    whole = gpu_eval(torch_cuda, plan, 0, n, bound=bound)
    inner = (prob.n_zones * (prob.n_types if not prob.mixed_types else
                             prob.n_types + prob.n_types * (prob.n_types - 1) // 2)
             * len(prob.mb_values) * len(prob.tp_values) * len(prob.dp_values))
    for piece in (inner - 1, max(inner // 3, 1), int(rng.integers(2 * inner, 9 * inner))):
        piece = max(piece, n // 300)  # (keeps the number of calls of the larger spaces bounded)
        parts = [gpu_eval(torch_cuda, plan, lo, min(piece, n - lo), bound=bound) for lo in range(0, n, piece)]
        for w, *ps in zip(whole, *parts):
            assert np.array_equal(w, np.concatenate(ps)), piece
    # ragged ends around whole shapes
    for _ in range(8):
        lo = int(rng.integers(0, n - 1))
        cnt = int(rng.integers(1, n - lo + 1))
        part = gpu_eval(torch_cuda, plan, lo, cnt, bound=bound)
        for w, q in zip(whole, part):
            assert np.array_equal(w[lo:lo + cnt], q), (lo, cnt)


def test_eval_batch_ragged_ranges_and_index_lists(case, torch_cuda):
    prob, plan, orc = case
    n = orc.num_candidates
    rng = np.random.default_rng(3)
    first, count = n // 3 + 1, min(n - n // 3 - 1, 1237)
    assert_eval_parity(gpu_eval(torch_cuda, plan, first, count),
                       orc.eval_batch(first, count))
    idx = rng.integers(0, n, 777).astype(np.uint64)
    assert_eval_parity(gpu_eval(torch_cuda, plan, 0, len(idx), indices=idx),
                       orc.eval_batch(indices=idx))
    # an out-of-range index inside a list is flagged, not evaluated
    bad = np.array([0, n, n - 1, 2 ** 40], np.uint64)
    t, c, m, k = gpu_eval(torch_cuda, plan, 0, 4, indices=bad)
    assert k[1] == k[3] == 0xFFFFFFFF and np.isinf(t[1]) and m[3] == 0
    assert k[0] == orc.eval_one(0).mask and k[2] == orc.eval_one(n - 1).mask
    # empty and out-of-range ranges
    plan.eval_batch(0, 0)
    from paper_2504_17096_amd.binding import SAILOR_ERANGE, SailorError
    with pytest.raises(SailorError) as ei:
        plan.eval_batch(n - 1, 2)
    assert ei.value.status == SAILOR_ERANGE


@pytest.mark.parametrize("objective", [MAX_THROUGHPUT, MIN_COST])
def test_best_plan_and_topk(case, torch_cuda, objective):
    prob, plan, orc = case
    stream = torch_cuda.cuda.current_stream().cuda_stream
    t, c, _, mask = orc.eval_batch(objective=objective, n_threads=THREADS)
    bounds = [None]
    ok = mask == 0
    if ok.any():
        val = c if objective == MAX_THROUGHPUT else 1.0 / t
        bounds += [off_data(float(np.median(val[ok]))), off_data(float(np.quantile(val[ok], 0.1))),
                   float(val[ok].min()) * (0.5 if objective == MAX_THROUGHPUT else 2.0)]
    for bound in bounds:
        want = orc.best(objective=objective, bound=bound, n_threads=THREADS)
        got = plan.best_plan(objective=objective, bound=bound, stream=stream)
        if want is None:
            assert got is None
        else:
            check_result(got, want, orc)
        for k in (1, 7, 64, 300):  # (above 128 the final ranking runs on several workgroups)
            want_k = orc.topk(k, objective=objective, bound=bound, n_threads=THREADS)
            got_k = plan.topk(k, objective=objective, bound=bound, stream=stream)
            check_topk(got_k, want_k, objective, orc, bound)
            if want_k:
                check_result(got_k[0], want_k[0], orc) if got_k[0].index == want_k[0].index else None
            if bound is not None:
                # With few pieces of the space alive under the bound the call above kept every
                # valid candidate of theirs in one pass; a plan that keeps minima for later calls
                # never does, so this one goes through the scan and its thresholds.
                plan.set_incremental(True)
                check_topk(plan.topk(k, objective=objective, bound=bound, stream=stream), want_k,
                           objective, orc, bound)
                plan.set_incremental(False)


def test_no_feasible_plan_and_availability_update(torch_cuda):
    prob = W.config1()
    plan, stream = _plan(prob), torch_cuda.cuda.current_stream().cuda_stream
    try:
        plan.set_avail(np.zeros_like(prob.avail))
        assert plan.best_plan(stream=stream) is None
        assert plan.topk(5, stream=stream) == []
        half = prob.avail // 2
        plan.set_avail(half)
        orc = Oracle(prob.with_avail(half))
        check_result(plan.best_plan(stream=stream), orc.best(), orc)
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, orc.num_candidates), orc.eval_batch())
    finally:
        plan.destroy()


def test_pieces_ruled_out_by_their_bounds_are_passed_over_and_nothing_is_lost(torch_cuda):
    # The bounds are taken at plan creation with the availability ignored (Sec. 4.2.1, H3, applied
    # to a piece of the space): a plan created while GPUs are scarce must still find what becomes
    # valid when many arrive, for every bound, and must pass over pieces only when a bound binds.
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = W.config2()
    scarce = np.minimum(prob.avail, 2)
    plan = _plan(prob.with_avail(scarce))
    try:
        ruled_out = 0
        for avail in (scarce, prob.avail, prob.avail * 4, prob.avail // 3):
            plan.set_avail(avail)
            orc = Oracle(prob.with_avail(avail))
            t, c, _, mask = orc.eval_batch(n_threads=THREADS)
            ok = mask == 0
            if not ok.any():
                assert plan.best_plan(stream=stream) is None
                continue
            for objective in (MAX_THROUGHPUT, MIN_COST):
                val = c if objective == MAX_THROUGHPUT else 1.0 / t
                lo, hi = float(val[ok].min()), float(val[ok].max())
                seen = []
                for q in (0.0, 0.02, 0.2, 0.6, 1.0):
                    # (for MIN_COST the bound is a floor on iterations/s: tight means large)
                    bound = off_data(lo + q * (hi - lo)) if objective == MAX_THROUGHPUT else \
                        off_data(hi - q * (hi - lo)) * (1.0 - 2e-7)
                    got = plan.topk(40, objective=objective, bound=bound, stream=stream)
                    seen.append(plan.last_scan())
                    check_topk(got, orc.topk(40, objective=objective, bound=bound, n_threads=THREADS),
                               objective, orc, bound)
                    want = orc.best(objective=objective, bound=bound, n_threads=THREADS)
                    best = plan.best_plan(objective=objective, bound=bound, stream=stream)
                    assert (best is None) == (want is None)
                    if want is not None:
                        check_result(best, want, orc)
                total = seen[0][1]
                evaluated = [e for e, _ in seen]
                assert evaluated == sorted(evaluated), evaluated  # a looser bound never rules out more
                ruled_out += evaluated[0] < total
        # (the bounds ignore the availability: where GPUs are scarce even the tightest bound that
        # leaves a plan may rule nothing out, with many GPUs it does)
        assert ruled_out >= 2, ruled_out
        # a budget below every plan's cost: nothing is evaluated, nothing is found
        assert plan.topk(40, objective=MAX_THROUGHPUT, bound=1e-30, stream=stream) == []
        assert plan.last_scan()[0] == 0
        # a bound that cannot bind, and no bound at all: every piece is evaluated
        plan.topk(40, objective=MAX_THROUGHPUT, bound=1e30, stream=stream)
        assert plan.last_scan()[0] == plan.last_scan()[1]
        plan.topk(40, objective=MAX_THROUGHPUT, stream=stream)
        assert plan.last_scan()[0] == plan.last_scan()[1]
    finally:
        plan.destroy()


def test_near_ties_follow_the_lowest_index_rule(torch_cuda):
    stream = torch_cuda.cuda.current_stream().cuda_stream
    for rel, first_wins in ((4e-6, True), (4e-5, False), (9.9e-6, True), (1.01e-5, False)):
        tf = np.zeros((2, 1, 1, 1)); tf[0] = 1e-3 * (1 + rel); tf[1] = 1e-3
        p = make_problem(n_layers=2, n_types=2, mb_list=(1,), tp_list=(1,), dp_list=(1,),
                         pp_list=[1], global_batch=4, t_fwd=tf, t_bwd=0.0, layer_params=0)
        plan, orc = _plan(p), Oracle(p)
        try:
            assert orc.best().index == (0 if first_wins else 1)
            assert plan.best_plan(stream=stream).index == orc.best().index
            assert [r.index for r in plan.topk(2, stream=stream)] == [1, 0]
        finally:
            plan.destroy()


def test_exact_duplicates_resolve_to_the_lowest_index(torch_cuda):
    # two zones with identical rows: mirrored plans have bit-identical keys
    stream = torch_cuda.cuda.current_stream().cuda_stream
    p = make_problem(n_layers=4, n_types=1, n_zones=2, max_segments=2, p2p=1_000_000,
                     bw=np.array([[1e10, 1e9], [1e9, 1e10]]), avail=8)
    plan, orc = _plan(p), Oracle(p)
    try:
        for objective in (MAX_THROUGHPUT, MIN_COST):
            check_result(plan.best_plan(objective=objective, stream=stream),
                         orc.best(objective=objective), orc)
            check_topk(plan.topk(16, objective=objective, stream=stream),
                       orc.topk(16, objective=objective), objective, orc)
    finally:
        plan.destroy()


def test_thousands_of_exact_ties_at_the_kth_place(torch_cuda):
    # 16 identical zones, equal links everywhere, no egress: every placement of a shape has
    # the same key, so the list to rank is far longer than k and only the index decides
    stream = torch_cuda.cuda.current_stream().cuda_stream
    p = make_problem(n_layers=4, n_types=1, n_zones=16, pp_list=[4], max_segments=3,
                     seg3_max_pp=4, mb_list=(1,), tp_list=(1,), dp_list=(1, 2), global_batch=8,
                     p2p=1_000_000, bw=1e9, avail=64)
    plan, orc = _plan(p), Oracle(p)
    try:
        assert orc.num_candidates > 20000
        for objective in (MAX_THROUGHPUT, MIN_COST):
            want = orc.topk(64, objective=objective)
            got = plan.topk(64, objective=objective, stream=stream)
            assert [r.index for r in got] == [e.index for e in want]
            check_result(plan.best_plan(objective=objective, stream=stream),
                         orc.best(objective=objective), orc)
    finally:
        plan.destroy()


def test_small_scratch_makes_topk_search_for_a_tighter_threshold(torch_cuda):
    # with room for only 100 survivors the first threshold (from the unit minima) overflows
    # and the library has to find one that keeps >= k candidates and fits
    from paper_2504_17096_amd.binding import SAILOR_ENOMEM, SailorError
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = W.config2()
    plan, orc = _plan(prob), Oracle(prob)
    try:
        plan.set_scratch(100, 4096)
        cheapest = orc.best(objective=MIN_COST)
        for objective, bound in ((MAX_THROUGHPUT, None), (MIN_COST, None),
                                 (MAX_THROUGHPUT, 1.5 * cheapest.cost)):
            check_topk(plan.topk(64, objective=objective, bound=bound, stream=stream),
                       orc.topk(64, objective=objective, bound=bound), objective, orc, bound)
            check_result(plan.best_plan(objective=objective, bound=bound, stream=stream),
                         orc.best(objective=objective, bound=bound), orc)
        # room for fewer survivors than k can never work: a clean error, not a crash
        plan.set_scratch(32, 4096)
        with pytest.raises(SailorError) as ei:
            plan.topk(64, stream=stream)
        assert ei.value.status == SAILOR_ENOMEM
        plan.set_scratch(1 << 16, 1 << 12)
        check_topk(plan.topk(64, stream=stream), orc.topk(64), MAX_THROUGHPUT, orc)
    finally:
        plan.destroy()


def test_one_pass_over_the_pieces_left_alive_falls_back_when_it_keeps_too_much(torch_cuda):
    # A bounded top-k query that leaves few pieces alive keeps all their valid candidates in one
    # pass.  More of them than the survivor buffer holds: the call goes through the scan and its
    # threshold instead.  More than half the buffer: this call stands, and the same query takes
    # the scan from the next call on.  The plans are the oracle's every time.
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = W.config2()
    orc = Oracle(prob)
    plan = _plan(prob)
    try:
        budget = 2.0 * orc.best(objective=MIN_COST).cost
        want = orc.topk(64, objective=MAX_THROUGHPUT, bound=budget, n_threads=THREADS)
        check_topk(plan.topk(64, objective=MAX_THROUGHPUT, bound=budget, stream=stream), want,
                   MAX_THROUGHPUT, orc, budget)
        live, total = plan.last_scan()
        kept = plan.last_counts()[0]
        t, c, _, mask = orc.eval_batch(n_threads=THREADS)
        n_within = int(np.count_nonzero((mask == 0) & (c <= budget)))
        # every plan within the budget was kept (the fp32 pass lets a hair more through)
        assert live <= 128 and live < total and n_within <= kept <= n_within * 1.01 + 10, (live, kept, n_within)
        assert kept > 1000  # (what the two cases below rely on)
        # half the buffer exceeded: the answer stands, the next call scans
        plan.set_scratch(kept + kept // 2, 4096)
        for rep in range(3):
            check_topk(plan.topk(64, objective=MAX_THROUGHPUT, bound=budget, stream=stream), want,
                       MAX_THROUGHPUT, orc, budget)
            assert (plan.last_counts()[0] == kept) == (rep == 0), (rep, plan.last_counts())
        # ... another query is tried in one pass again
        other = 1.9 * orc.best(objective=MIN_COST).cost
        check_topk(plan.topk(64, objective=MAX_THROUGHPUT, bound=other, stream=stream),
                   orc.topk(64, objective=MAX_THROUGHPUT, bound=other, n_threads=THREADS),
                   MAX_THROUGHPUT, orc, other)
        # the buffer exceeded: the scan's threshold decides within the same call
        plan.set_scratch(kept // 2, 4096)
        for q, w in ((budget, want), (other, None)):
            w = w or orc.topk(64, objective=MAX_THROUGHPUT, bound=q, n_threads=THREADS)
            check_topk(plan.topk(64, objective=MAX_THROUGHPUT, bound=q, stream=stream), w,
                       MAX_THROUGHPUT, orc, q)
            assert plan.last_counts()[0] <= kept // 2
    finally:
        plan.destroy()


def test_ties_that_overflow_the_re_evaluated_list_give_a_clean_error(torch_cuda):
    # thousands of exact ties lie inside the rounding band of the k-th key; with room for only
    # 40 re-evaluated records the call must report SAILOR_ENOMEM (and rank nothing), and work
    # again once the room is back
    from paper_2504_17096_amd.binding import SAILOR_ENOMEM, SailorError
    stream = torch_cuda.cuda.current_stream().cuda_stream
    p = make_problem(n_layers=4, n_types=1, n_zones=16, pp_list=[4], max_segments=3,
                     seg3_max_pp=4, mb_list=(1,), tp_list=(1,), dp_list=(1, 2), global_batch=8,
                     p2p=1_000_000, bw=1e9, avail=64)
    plan, orc = _plan(p), Oracle(p)
    try:
        plan.set_scratch(1 << 16, 40)
        for k in (64, 200):  # ranked by one workgroup / by several
            with pytest.raises(SailorError) as ei:
                plan.topk(k, stream=stream)
            assert ei.value.status == SAILOR_ENOMEM
        with pytest.raises(SailorError) as ei:
            plan.best_plan(stream=stream)
        assert ei.value.status == SAILOR_ENOMEM
        plan.set_scratch(1 << 16, 1 << 15)
        assert [r.index for r in plan.topk(64, stream=stream)] == [e.index for e in orc.topk(64)]
        check_result(plan.best_plan(stream=stream), orc.best(), orc)
    finally:
        plan.destroy()


@pytest.mark.parametrize("seed", range(100, 124))
def test_random_small_problems(torch_cuda, seed):
    # shapes drawn at random: odd pool counts, deep pipelines on few layers, batches that
    # some (D, mb) pairs do not divide, empty pools
    rng = np.random.default_rng(seed)
    n_layers = int(rng.choice([3, 4, 5, 6, 8, 9, 12]))
    prob = W.tiny_problem(seed, n_layers=n_layers, n_types=int(rng.integers(1, 4)),
                          n_zones=int(rng.integers(1, 4)), max_segments=int(rng.integers(1, 4)),
                          seg3_max_pp=int(rng.choice([3, 4, 6, 12])),
                          uniform_layers=bool(rng.integers(0, 2)),
                          partitions_per_pp=int(rng.integers(1, 4)),
                          with_egress=bool(rng.integers(0, 2)))
    prob.global_batch = int(rng.choice([8, 12, 16, 24]))
    prob.per_segment_tp = bool(seed % 2)
    if seed % 3 == 0:
        prob = prob.with_bw_poly(W.bandwidth_poly(prob, seed))
    if seed % 4 == 1:
        prob = prob.with_mixed_types()
    avail = prob.avail.copy()
    avail[rng.random(avail.shape) < 0.25] = 0
    prob = prob.with_avail(avail)
    plan, orc = _plan(prob), Oracle(prob)
    stream = torch_cuda.cuda.current_stream().cuda_stream
    try:
        n = orc.num_candidates
        assert plan.num_candidates() == n
        want = orc.eval_batch(n_threads=THREADS)
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, n), want)
        idx = rng.integers(0, n, 500).astype(np.uint64)
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, len(idx), indices=idx),
                           orc.eval_batch(indices=idx))
        for objective in (MAX_THROUGHPUT, MIN_COST):
            ok = want[3] == 0
            bounds = [None]
            if ok.any():
                val = want[1] if objective == MAX_THROUGHPUT else 1.0 / want[0]
                bounds.append(off_data(float(np.quantile(val[ok], 0.3))))
            for bound in bounds:
                w_best = orc.best(objective=objective, bound=bound, n_threads=THREADS)
                g_best = plan.best_plan(objective=objective, bound=bound, stream=stream)
                if w_best is None:
                    assert g_best is None
                else:
                    check_result(g_best, w_best, orc)
                check_topk(plan.topk(17, objective=objective, bound=bound, stream=stream),
                           orc.topk(17, objective=objective, bound=bound, n_threads=THREADS),
                           objective, orc, bound)
    finally:
        plan.destroy()


def test_widest_lists_with_a_tp_digit_per_segment(torch_cuda):
    # 64 pools, 8 TP degrees per segment: ~5e7 candidates; sampled outputs and selections
    prob = wide_problem().with_per_segment_tp()
    plan, orc = _plan(prob), Oracle(prob)
    stream = torch_cuda.cuda.current_stream().cuda_stream
    try:
        n = orc.num_candidates
        assert plan.num_candidates() == n > 4e7
        rng = np.random.default_rng(8)
        idx = rng.integers(0, n, 200000).astype(np.uint64)
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, len(idx), indices=idx),
                           orc.eval_batch(indices=idx, n_threads=THREADS))
        first = n - 3_000_001
        assert_eval_parity(gpu_eval(torch_cuda, plan, first, 3_000_001),
                           orc.eval_batch(first, 3_000_001, n_threads=THREADS))
        for objective in (MAX_THROUGHPUT, MIN_COST):
            check_result(plan.best_plan(objective=objective, stream=stream),
                         orc.best(objective=objective, n_threads=THREADS), orc)
            check_topk(plan.topk(64, objective=objective, stream=stream),
                       orc.topk(64, objective=objective, n_threads=THREADS), objective, orc)
    finally:
        plan.destroy()


def test_seventy_five_pools_five_zones_five_types_with_pairs(torch_cuda):
    # 5 zones x (5 types + 10 pairs) = 75 pools: beyond one 64-bit word of pool relations
    prob = W.tiny_problem(8, n_layers=4, n_types=5, n_zones=5, max_segments=2, partitions_per_pp=2).with_mixed_types()
    plan, orc = _plan(prob), Oracle(prob)
    stream = torch_cuda.cuda.current_stream().cuda_stream
    try:
        n = orc.num_candidates
        assert plan.num_candidates() == n and n > 1_000_000
        first, count = n - 1_500_003, 1_500_003           # two-segment blocks, a ragged range
        assert_eval_parity(gpu_eval(torch_cuda, plan, first, count), orc.eval_batch(first, count, n_threads=THREADS))
        idx = np.random.default_rng(75).integers(0, n, 300_000).astype(np.uint64)
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, len(idx), indices=idx),
                           orc.eval_batch(indices=idx, n_threads=THREADS))
        for objective in (MAX_THROUGHPUT, MIN_COST):
            check_topk(plan.topk(64, objective=objective, stream=stream),
                       orc.topk(64, objective=objective, n_threads=THREADS), objective, orc)
            check_result(plan.best_plan(objective=objective, stream=stream),
                         orc.best(objective=objective, n_threads=THREADS), orc)
        # three segments on 75 pools as well, on a smaller model
        p3 = W.tiny_problem(9, n_layers=3, n_types=5, n_zones=5, max_segments=3, seg3_max_pp=3,
                            partitions_per_pp=1).with_mixed_types()
        plan3, orc3 = _plan(p3), Oracle(p3)
        try:
            n3 = orc3.num_candidates
            idx = np.random.default_rng(76).integers(0, n3, 400_000).astype(np.uint64)
            assert_eval_parity(gpu_eval(torch_cuda, plan3, 0, len(idx), indices=idx),
                               orc3.eval_batch(indices=idx, n_threads=THREADS))
            assert_eval_parity(gpu_eval(torch_cuda, plan3, n3 - 700_001, 700_001),
                               orc3.eval_batch(n3 - 700_001, 700_001, n_threads=THREADS))
            check_topk(plan3.topk(32, stream=stream), orc3.topk(32, n_threads=THREADS), MAX_THROUGHPUT, orc3)
        finally:
            plan3.destroy()
    finally:
        plan.destroy()


def test_eval_batch_replays_from_a_captured_graph(torch_cuda):
    # sailor_eval_batch only enqueues kernels on the caller's stream (no host synchronisation,
    # no memset), so it can be captured; every replay must reproduce the eager outputs
    torch = torch_cuda
    prob = W.config2()
    plan, orc = _plan(prob), Oracle(prob)
    try:
        n = orc.num_candidates
        want = orc.eval_batch()
        eager = gpu_eval(torch, plan, 0, n)
        dev = "cuda:0"
        t = torch.zeros(n, dtype=torch.float32, device=dev)
        c = torch.zeros(n, dtype=torch.float32, device=dev)
        m = torch.zeros(n, dtype=torch.int64, device=dev)
        k = torch.zeros(n, dtype=torch.int32, device=dev)
        idx = torch.from_numpy(np.random.default_rng(1).integers(0, n, 4096).astype(np.int64)).to(dev)
        ti = torch.zeros(4096, dtype=torch.float32, device=dev)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            plan.eval_batch(0, n, d_time=t, d_cost=c, d_mem=m, d_mask=k, stream=side.cuda_stream)  # warm
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                plan.eval_batch(0, n, d_time=t, d_cost=c, d_mem=m, d_mask=k, stream=side.cuda_stream)
                plan.eval_batch(0, 4096, d_indices=idx, d_time=ti, stream=side.cuda_stream)
        torch.cuda.current_stream().wait_stream(side)
        for rep in range(3):
            for x in (t, c, m, k, ti):
                x.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = (t.cpu().numpy(), c.cpu().numpy(), m.cpu().numpy().view(np.uint64),
                   k.cpu().numpy().view(np.uint32))
            for a, b in zip(got, eager):
                assert np.array_equal(a, b), rep
            assert np.array_equal(ti.cpu().numpy(), eager[0][idx.cpu().numpy()])
            assert_eval_parity(got, want)
            # eager work of the program between the replays
            assert plan.best_plan().index == orc.best().index
    finally:
        plan.destroy()


@pytest.mark.parametrize("mixed", [False, True])
def test_calls_captured_while_a_new_availability_is_due(torch_cuda, mixed):
    # replays read the table that the host holds at the time; calls outside the graph see it too, before
    # the first replay and behind a replay that has brought it to the device (kept minima included)
    torch = torch_cuda
    prob = W.config2()
    if mixed:
        prob = W.tiny_problem(77, n_layers=6, n_types=2, n_zones=2, max_segments=3, seg3_max_pp=6,
                              partitions_per_pp=2).with_mixed_types()
    rng = np.random.default_rng(4)
    tables = [np.where(rng.random(prob.avail.shape) < 0.2, 0, rng.integers(1, prob.avail.max() + 1, prob.avail.shape))
              .astype(np.int32) for _ in range(8)]
    orcs = [Oracle(prob.with_avail(a)) for a in tables]
    plan, kept = _plan(prob), _plan(prob)
    kept.set_incremental(True)
    try:
        n, dev = orcs[0].num_candidates, "cuda:0"
        out = [torch.zeros(n, dtype=d, device=dev) for d in (torch.float32, torch.float32, torch.int64, torch.int32)]
        idx = torch.from_numpy(rng.integers(0, n, 4096)).to(dev)
        ti = torch.zeros(4096, dtype=torch.float32, device=dev)
        side = torch.cuda.Stream()
        st = side.cuda_stream
        side.wait_stream(torch.cuda.current_stream())

        def calls():
            for p in (plan, kept):
                p.eval_batch(0, n, d_time=out[0], d_cost=out[1], d_mem=out[2], d_mask=out[3], stream=st)
                p.eval_batch(0, 4096, d_indices=idx, d_time=ti, stream=st)

        def best(p, orc):
            got, want = p.best_plan(stream=st), orc.best(n_threads=THREADS)
            assert (got is None) == (want is None)
            if want is not None:
                check_result(got, want, orc)

        with torch.cuda.stream(side):
            calls()
            side.synchronize()
            for p in (plan, kept):
                p.set_avail(tables[0])
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                calls()
        best(plan, orcs[0])
        best(kept, orcs[0])
        for table, orc in zip(tables, orcs):
            torch.cuda.synchronize()  # the replays have finished
            for p in (plan, kept):
                p.set_avail(table)
            for x in (*out, ti):
                x.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = (out[0].cpu().numpy(), out[1].cpu().numpy(), out[2].cpu().numpy().view(np.uint64),
                   out[3].cpu().numpy().view(np.uint32))
            assert_eval_parity(got, orc.eval_batch(n_threads=THREADS))
            assert np.array_equal(ti.cpu().numpy(), got[0][idx.cpu().numpy()])
            best(plan, orc)
            best(kept, orc)
    finally:
        plan.destroy()
        kept.destroy()


@pytest.mark.parametrize("pps,n_shapes", [([2, 8, 64], 2048), ([1, 2, 8, 64], 2049)])
def test_index_lists_where_the_shapes_leave_lds(torch_cuda, pps, n_shapes):
    # the stages of up to 2 048 shapes lie in LDS, those of more are read from memory
    L, rng = 64, np.random.default_rng(6)
    shape = (2, 2, 2, L)
    fwd = rng.uniform(0.5e-3, 2e-3, shape)
    prob = make_problem(n_layers=L, n_types=2, n_zones=2, mb_list=(1, 2), tp_list=(1, 2), dp_list=(1, 2, 4), pp_list=pps,
                        max_segments=3, seg3_max_pp=64, global_batch=32, uniform_layers=False, t_fwd=fwd, t_bwd=2 * fwd,
                        t_upd=1e-5, layer_params=rng.integers(1_000_000, 90_000_000, L), act=3_000_000, p2p=2_000_000,
                        cap=np.array([8, 3], np.uint64) * np.uint64(1 << 30), node=np.array([2, 1]),
                        avail=np.array([[120, 60], [40, 250]]), bw=np.array([[1e10, 1e9], [2e9, 1e10]]),
                        price=np.array([3.0, 1.5]), egress=np.array([[0, 2e-11], [1e-11, 0]]))
    cuts = sum(1 + (p - 1) + (p - 1) * (p - 2) // 2 for p in pps)
    assert cuts == n_shapes
    plan, orc = _plan(prob), Oracle(prob)
    try:
        n = orc.num_candidates
        assert plan.num_candidates() == n
        idx = np.concatenate([rng.integers(0, n, 200_000), [0, n - 1]]).astype(np.uint64)
        want = orc.eval_batch(indices=idx, n_threads=THREADS)
        assert len(set((want[3] & 15).tolist())) > 4
        assert_eval_parity(gpu_eval(torch_cuda, plan, 0, len(idx), indices=idx), want)
    finally:
        plan.destroy()


def test_independent_plans_serve_two_host_threads(torch_cuda):
    # one plan per thread, each on a stream of its own: the calls overlap in time (ctypes
    # releases the interpreter lock) and every one must return what the oracle selects
    import threading
    torch = torch_cuda
    probs = [W.config2(), W.config1().with_per_segment_tp()]
    orcs = [Oracle(p) for p in probs]
    want = [(o.best(MAX_THROUGHPUT), o.topk(16, MIN_COST)) for o in orcs]
    plans = [_plan(p) for p in probs]
    streams = [torch.cuda.Stream() for _ in probs]
    errors = []

    def serve(i):
        try:
            for rep in range(40):
                best = plans[i].best_plan(MAX_THROUGHPUT, stream=streams[i].cuda_stream)
                assert best.index == want[i][0].index, (i, rep)
                top = plans[i].topk(16, MIN_COST, stream=streams[i].cuda_stream)
                assert [r.index for r in top] == [e.index for e in want[i][1]], (i, rep)
        except BaseException as e:  # reported by the main thread
            errors.append(e)

    try:
        workers = [threading.Thread(target=serve, args=(i,)) for i in range(len(probs))]
        for w in workers:
            w.start()
        for w in workers:
            w.join(timeout=100)
        assert not any(w.is_alive() for w in workers)
        assert not errors, errors
        torch.cuda.synchronize()
    finally:
        for p in plans:
            p.destroy()


def test_calls_of_one_plan_move_between_streams(torch_cuda):
    # nothing orders the streams, and a call returns while its last kernel is retiring (the more so on a
    # GPU that another plan keeps busy): what still runs of it must leave the counters of the plan's later
    # calls alone.  Few and many survivors in turn: up to 64 are one workgroup's, more are shared by all
    torch = torch_cuda
    prob = make_problem(n_layers=8, n_types=8, n_zones=2, mb_list=(1, 2), tp_list=(1, 2), dp_list=(1, 2, 4),
                        pp_list=[1, 4], max_segments=2, layer_params=1_000_000, act=1_000_000,
                        price=np.arange(1.0, 9.0), bw=1e10)
    plan, orc, busy = _plan(prob), Oracle(prob), _plan(W.config2())
    try:
        cheapest = orc.best(MIN_COST)
        budget = cheapest.cost * (1 + 1e-6)
        best = {None: orc.best(), budget: orc.best(MAX_THROUGHPUT, budget)}
        top = orc.topk(8, MIN_COST)
        streams = [torch.cuda.Stream() for _ in range(3)]
        n = busy.num_candidates()
        out = torch.empty(n, dtype=torch.float32, device="cuda:0")
        torch.cuda.synchronize()
        counts, rng = {None: set(), budget: set()}, np.random.default_rng(5)
        for rep in range(300):
            if rep % 10 == 0:
                for _ in range(10):
                    busy.eval_batch(0, n, d_time=out, stream=streams[2].cuda_stream)
            st = streams[int(rng.integers(2))].cuda_stream
            if rng.integers(4) == 0:
                check_topk(plan.topk(8, MIN_COST, stream=st), top, MIN_COST, orc)
                continue
            bound = (None, budget)[int(rng.integers(2))]
            check_result(plan.best_plan(MAX_THROUGHPUT, bound, stream=st), best[bound], orc)
            counts[bound].add(plan.last_counts()[1:])
        torch.cuda.synchronize()
        # (the candidates within the tie band of the minimum do not depend on the order of the scan)
        assert len(counts[None]) == len(counts[budget]) == 1, counts
        assert min(counts[None])[0] > 64 >= max(counts[budget])[0] > 0
    finally:
        plan.destroy()
        busy.destroy()


def test_timing_modes_report_the_scan_and_the_whole_call(torch_cuda):
    from paper_2504_17096_amd.binding import SAILOR_EINVAL, SailorError
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = W.config2()
    plan = _plan(prob)
    try:
        want = plan.best_plan(stream=stream).index
        with pytest.raises(SailorError) as ei:   # nothing was recorded in mode 0
            plan.last_timing()
        assert ei.value.status == SAILOR_EINVAL
        plan.set_timing(1)
        assert plan.best_plan(stream=stream).index == want
        total, scan = plan.last_timing()
        assert total == 0.0 and 0.0 < scan < 50.0
        plan.set_timing(2)
        assert [r.index for r in plan.topk(3, stream=stream)][0] == want
        total, scan2 = plan.last_timing()
        assert 0.0 < scan2 <= total < 50.0
        n = plan.num_candidates()
        t = torch_cuda.empty(n, dtype=torch_cuda.float32, device="cuda:0")
        plan.eval_batch(0, n, d_time=t, stream=stream)
        assert 0.0 < plan.last_timing()[1] < 50.0
        plan.set_timing(0)
        assert plan.best_plan(stream=stream).index == want
        with pytest.raises(SailorError):
            plan.last_timing()
        with pytest.raises(SailorError):
            plan.set_timing(3)
    finally:
        plan.destroy()


@pytest.mark.parametrize("parts", [2, 5])
@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg2_mixed", "tiny4_segtp", "wide"])
def test_selection_with_every_scan_unit_cut_into_parts(torch_cuda, name, parts):
    # units that run long are cut by measured time at plan creation, which small problems
    # never trigger: sailor_set_scan_unit_parts cuts every unit, and the selections (scan,
    # unit list, collect pass over the listed parts) must not change
    from paper_2504_17096_amd.binding import set_scan_unit_parts
    prob = PROBLEMS[name]()
    set_scan_unit_parts(parts)
    try:
        plan, orc = _plan(prob), Oracle(prob)
    finally:
        set_scan_unit_parts(0)
    stream = torch_cuda.cuda.current_stream().cuda_stream
    try:
        cheapest = orc.best(objective=MIN_COST, n_threads=THREADS)
        for objective, bound in ((MAX_THROUGHPUT, None), (MIN_COST, None),
                                 (MAX_THROUGHPUT, 1.3 * cheapest.cost)):
            check_result(plan.best_plan(objective=objective, bound=bound, stream=stream),
                         orc.best(objective=objective, bound=bound, n_threads=THREADS), orc)
            for k in (5, 64, 300):
                check_topk(plan.topk(k, objective=objective, bound=bound, stream=stream),
                           orc.topk(k, objective=objective, bound=bound, n_threads=THREADS),
                           objective, orc, bound)
    finally:
        plan.destroy()


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n_dp", [1, 4, 7, 8])
def test_scan_at_the_edges_of_its_lane_space(torch_cuda, n_dp, mixed):
    # three mb x n_dp degrees x six pools (five with three segments; nine and eight with pairs of types)
    # in chunks of 64 lanes, walked from the last one down: 15 to 216 of them, 54 and 60 (one short
    # chunk), 72 (a second of eight), 126, 192 (three whole ones); waves without a chunk, plans dropped
    # on their leading segments.  Tight, loose and no bounds; fp64 values against the oracle's, 1e-9.
    from dataclasses import replace
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = replace(W.tiny_problem(72, n_layers=8, n_zones=3, seg3_max_pp=8), global_batch=3360,
                   dp_values=np.arange(1, n_dp + 1, dtype=np.int32))
    prob = prob.with_mixed_types() if mixed else prob
    plan, orc = _plan(prob), Oracle(prob)
    try:
        t, c, _, mask = orc.eval_batch(n_threads=THREADS)
        ok = mask == 0
        assert ok.any()
        for objective in (MAX_THROUGHPUT, MIN_COST):
            val = c if objective == MAX_THROUGHPUT else 1.0 / t
            lo, hi = float(val[ok].min()), float(val[ok].max())
            for bound in (None, off_data(lo + 0.02 * (hi - lo)), off_data(lo + 0.6 * (hi - lo))):
                check_result(plan.best_plan(objective=objective, bound=bound, stream=stream),
                             orc.best(objective=objective, bound=bound, n_threads=THREADS), orc)
                for k in (1, 64):
                    check_topk(plan.topk(k, objective=objective, bound=bound, stream=stream),
                               orc.topk(k, objective=objective, bound=bound, n_threads=THREADS),
                               objective, orc, bound)
    finally:
        plan.destroy()


@pytest.mark.parametrize("form", ["distinct", "ties", "scarce"])
def test_threshold_among_more_units_than_a_workgroup_keeps(torch_cuda, form):
    # 290 shapes x a TP degree per segment: over 8 192 units, whose k-th smallest minimum is found by rank
    # (distinct times), by its digits (identical layers and pools: thousands of equal minima), or is not
    # there (fewer valid units than k); k on both sides of the 128 that the ranks are taken up to
    L, rng = 24, np.random.default_rng(3)
    shape = (2, 1, 4, L)
    fwd = np.full(shape, 1e-3) if form == "ties" else rng.uniform(0.5e-3, 2e-3, shape)
    prob = make_problem(n_layers=L, n_types=2, n_zones=2, mb_list=(1,), tp_list=(1, 2, 4, 8), dp_list=(1, 2),
                        pp_list=[1, 2, 24], max_segments=3, seg3_max_pp=24, global_batch=64, uniform_layers=False,
                        t_fwd=fwd, t_bwd=2 * fwd, layer_params=1_000_000, act=1_000_000, p2p=1_000_000,
                        avail=np.array([[24, 0], [0, 3]]) if form == "scarce" else np.full((2, 2), 400),
                        bw=np.array([[1e10, 1e9], [1e9, 1e10]])).with_per_segment_tp(True)
    plan, orc = _plan(prob), Oracle(prob)
    try:
        assert plan.num_candidates() == orc.num_candidates
        for k in (1, 17, 64, 65, 128, 129):
            check_topk(plan.topk(k), orc.topk(k, n_threads=4), MAX_THROUGHPUT, orc)
        # the units that the plan keeps: beyond what the digit form holds in registers, and where the values
        # are distinct beyond what the rank form holds, too (pools without room take units away)
        assert plan.last_scan()[1] > (8192 if form == "scarce" else 16384)
    finally:
        plan.destroy()


@pytest.mark.parametrize("mixed, zones, parts", [(False, 1, 40), (False, 2, 40), (True, 1, 40), (True, 2, 40), (True, 1, 1),
                                                 (True, 2, 1)])
def test_scan_guided_by_a_running_limit(torch_cuda, mixed, zones, parts):
    # More units than fit on the chip at once: the first of their order are shared by workgroups, the others
    # wait for them and take several units each.  The order is that of the availability at creation, so it is
    # set to one that rules the best units out (and nothing, and everything); one zone, where neighbouring
    # segments cannot share a type; degrees that pairs of types cannot halve (1, 3); k on both sides of
    # what the running k-th key is kept for (128), and of the plans there are.  Whole units of pairs of types: fewer,
    # which do fit, and guide the best plan's scan only.  Against the oracle, whole numbers and indices the same.
    from dataclasses import replace
    from paper_2504_17096_amd.binding import set_scan_unit_parts
    stream = torch_cuda.cuda.current_stream().cuda_stream
    prob = replace(W.tiny_problem(73, n_layers=8, n_zones=zones, seg3_max_pp=8), global_batch=768,
                   dp_values=np.array([1, 2, 3, 4, 8], np.int32)).with_per_segment_tp(True).with_mixed_types(mixed)
    set_scan_unit_parts(parts)
    try:
        plan = _plan(prob.with_avail(np.minimum(prob.avail, 2)))
    finally:
        set_scan_unit_parts(0)
    try:
        for avail in (np.minimum(prob.avail, 2), prob.avail * 4, np.zeros_like(prob.avail), prob.avail):
            plan.set_avail(avail)
            orc = Oracle(prob.with_avail(avail))
            t, c, _, mask = orc.eval_batch(n_threads=THREADS)
            ok = mask == 0
            for objective in (MAX_THROUGHPUT, MIN_COST):
                val = (c if objective == MAX_THROUGHPUT else 1.0 / t)[ok]
                for bound in (None, off_data(float(np.median(val))) if ok.any() else 1.0):
                    best = plan.best_plan(objective=objective, bound=bound, stream=stream)
                    want = orc.best(objective=objective, bound=bound, n_threads=THREADS)
                    assert (best is None) == (want is None)
                    if want is not None:
                        check_result(best, want, orc)
                    for k in (1, 128, 129):
                        check_topk(plan.topk(k, objective=objective, bound=bound, stream=stream),
                                   orc.topk(k, objective=objective, bound=bound, n_threads=THREADS),
                                   objective, orc, bound)
        # units: more than the chip's 8 192 waves, and twice that for a k-th key; pairs of types: more than 512 waves
        assert plan.last_scan()[1] > 16384 if parts > 1 else 512 < plan.last_scan()[1] < 8192
    finally:
        plan.destroy()


@pytest.mark.parametrize("objective", [MAX_THROUGHPUT, MIN_COST])
def test_more_ties_than_the_first_survivor_buffers_hold(torch_cuda, objective):
    # 16 zones that do not differ: 77 296 placements of eight stages in up to three segments tie for the best,
    # and the buffers a plan starts with (64 Ki kept, 16 Ki re-evaluated) are enlarged by the first query
    Z = 16
    prob = make_problem(n_layers=8, n_zones=Z, mb_list=(1,), tp_list=(1,), dp_list=(1, 2), pp_list=[8], max_segments=3,
                        seg3_max_pp=8, global_batch=32, avail=np.full((Z, 1), 64), bw=np.full((Z, Z), 1e10), p2p=1_000_000)
    orc = Oracle(prob)
    for first in ("best", "topk"):
        plan = _plan(prob)
        try:
            for call in (("best", "topk") if first == "best" else ("topk", "best")):
                if call == "best":
                    check_result(plan.best_plan(objective=objective), orc.best(objective, n_threads=4), orc)
                else:
                    check_topk(plan.topk(64, objective=objective), orc.topk(64, objective, n_threads=4), objective, orc)
                assert plan.last_counts()[0] > 1 << 16
        finally:
            plan.destroy()


@pytest.mark.parametrize("k", [65, 128])
def test_one_degree_left_to_a_budget_fills_the_slots_of_the_kth_key(torch_cuda, k):
    # 416 pieces of four waves each; the batch leaves one data-parallel degree of eight, so 60 plans of a piece's
    # lane space, all of them the first wave's.  Whatever wave they lie in, 416 pieces name 256 keys, of which the
    # k-th bounds what is kept: some thousands at most, of 120 000 valid plans.  (64 of the slots were within reach.)
    rng = np.random.default_rng(31)
    G, Z, L, mb = 3, 4, 12, (1, 2, 4, 8, 16)
    splits = {p: [np.diff([0, *sorted(rng.choice(np.arange(1, L), p - 1, replace=False)), L]).tolist() for _ in range(8)]
              for p in (2, 3, 4, 6)}
    bw = rng.uniform(0.5e9, 2e9, (Z, Z))
    np.fill_diagonal(bw, rng.uniform(0.8e10, 1.2e10, Z))
    prob = make_problem(
        n_layers=L, n_types=G, n_zones=Z, mb_list=mb, tp_list=(1, 2), dp_list=(7, 8, 9, 11, 13, 17, 19, 23),
        pp_list=[2, 3, 4, 6], partitions=splits, global_batch=128, max_segments=2,
        t_fwd=rng.uniform(0.5e-3, 3e-3, (G, 5, 2, 1)), t_bwd=rng.uniform(1e-3, 5e-3, (G, 5, 2, 1)),
        p2p=rng.integers(1_000_000, 9_000_000, 5).astype(np.uint64), cap=1 << 40, price=rng.uniform(0.5, 4.0, G),
        avail=10_000, bw=bw)
    orc, plan = Oracle(prob), _plan(prob)
    try:
        t, c, _, mask = orc.eval_batch(n_threads=THREADS)
        ok = mask == 0
        assert ok.sum() > 100_000
        for objective in (MAX_THROUGHPUT, MIN_COST):
            # a bound that all plans meet
            bound = 2.0 * float(c[ok].max()) if objective == MAX_THROUGHPUT else 0.5 / float(t[ok].max())
            check_topk(plan.topk(k, objective=objective, bound=bound), orc.topk(k, objective, bound=bound, n_threads=THREADS),
                       objective, orc, bound)
            assert plan.last_scan()[1] == 416
            assert k <= plan.last_counts()[0] < ok.sum() // 8
    finally:
        plan.destroy()


@pytest.mark.parametrize("objective", [MAX_THROUGHPUT, MIN_COST])
def test_a_guided_scan_that_finds_nothing_waits_once(torch_cuda, objective):
    # 9.2e8 plans; what is available is of a type that holds no stage, which no bound of a piece knows.  A workgroup
    # takes six pieces, and four times as many where each is cut in four.  It waits up to 8 us for the first ones to
    # find something; what it takes longer for a further piece is less than that, since it does not wait again.
    from dataclasses import replace
    from paper_2504_17096_amd.binding import set_scan_unit_parts
    prob = W.config4()
    reserved = prob.mem_reserved.copy()
    reserved[-1] = prob.mem_capacity[-1]
    prob = replace(prob, mem_reserved=reserved).with_per_segment_tp(True)
    avail = prob.avail * (np.arange(prob.n_types) == prob.n_types - 1)
    pieces, took = [], []
    for parts in (1, 4):
        set_scan_unit_parts(parts)
        try:
            plan = _plan(prob)
        finally:
            set_scan_unit_parts(0)
        try:
            assert plan.best_plan(objective=objective) is not None
            pieces.append(-(-plan.last_scan()[1] * 3 // 8192))  # workgroups of three waves, 8 192 waves at once
            plan.set_avail(avail)
            plan.set_timing(1)
            times = []
            for _ in range(12):
                assert plan.topk(64, objective=objective) == []
                times.append(plan.last_timing()[1])
            took.append(min(times))
            assert plan.best_plan(objective=objective) is None
        finally:
            plan.destroy()
    assert pieces[1] >= pieces[0] + 12
    assert took[1] - took[0] < (pieces[1] - pieces[0]) * 0.008, (pieces, took)


@pytest.mark.parametrize("make, parts", [
    (lambda: wide_problem(5), 40),   # 64 pools, 24 degrees; one and two segments
    (lambda: W.tiny_problem(75, n_layers=3, n_types=4, n_zones=7, seg3_max_pp=3, partitions_per_pp=1).with_mixed_types(), 60),  # 70 pools
])
def test_scans_without_a_limit_take_the_longest_units_first(torch_cuda, make, parts):
    # more units than fit on the chip at once, in an order of their own: every one is scanned, once.  k above
    # what a running key is kept for, a k behind which nothing valid is left, and minima that are kept while the
    # availability, by which they were ordered, changes.
    from paper_2504_17096_amd.binding import set_scan_unit_parts
    prob = make()
    set_scan_unit_parts(parts)
    try:
        plan = _plan(prob)
    finally:
        set_scan_unit_parts(0)
    try:
        for avail in (np.minimum(prob.avail, 3), prob.avail):
            plan.set_avail(avail)
            orc = Oracle(prob.with_avail(avail))
            t, c, _, mask = orc.eval_batch(n_threads=THREADS)
            for objective in (MAX_THROUGHPUT, MIN_COST):
                val = (c if objective == MAX_THROUGHPUT else 1.0 / t)[mask == 0]
                for bound in (None, off_data(float(np.median(val)))):
                    for k in (129, 4096) if bound is None else (129,):
                        check_topk(plan.topk(k, objective=objective, bound=bound),
                                   orc.topk(k, objective=objective, bound=bound, n_threads=THREADS), objective, orc, bound)
                    assert plan.last_scan()[1] * 2 > 8192
                want = orc.best(objective=objective, n_threads=THREADS)
                for on in (True, True, False):
                    plan.set_incremental(on)
                    check_result(plan.best_plan(objective=objective), want, orc)
    finally:
        plan.destroy()


def _many_small_units(n_zones, mixed, max_segments):
    """More whole units of two waves than twice the chip's 8 192 waves, of few plans each: a TP degree per segment, and
    many layer splits of one depth.  With two segments the lane space takes three rounds of a workgroup (eight
    microbatch sizes, 24 degrees, two pools), with three it is less than a wave."""
    rng = np.random.default_rng(100 + max_segments)
    L, G, tp = 24, 2 if max_segments == 3 else 1, (1, 2, 4, 8)
    P, n_splits = (8, 8) if max_segments == 3 else (12, 48)
    mb, dp = ((1,), (1, 2)) if max_segments == 3 else (
        (1, 2, 3, 4, 6, 8, 12, 24), (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16, 18, 20, 21, 24, 28, 30, 35, 36, 40, 42))
    splits = set()
    while len(splits) < n_splits:
        splits.add(tuple(np.diff([0, *sorted(rng.choice(np.arange(1, L), P - 1, replace=False)), L]).tolist()))
    bw = rng.uniform(0.5e9, 2e9, (n_zones, n_zones))
    np.fill_diagonal(bw, rng.uniform(0.8e10, 1.2e10, n_zones))
    prob = make_problem(
        n_layers=L, n_types=G, n_zones=n_zones, mb_list=mb, tp_list=tp, dp_list=dp, pp_list=[P],
        partitions={P: [list(s) for s in sorted(splits)]}, global_batch=24 * 5040, max_segments=max_segments,
        seg3_max_pp=P, uniform_layers=False, t_fwd=rng.uniform(0.5e-3, 3e-3, (G, len(mb), 4, L)),
        t_bwd=rng.uniform(1e-3, 5e-3, (G, len(mb), 4, L)), t_upd=rng.uniform(1e-4, 3e-4, (G, 4, L)),
        act=rng.integers(10_000_000, 400_000_000, (len(mb), 4)).astype(np.uint64),
        p2p=rng.integers(1_000_000, 9_000_000, len(mb)).astype(np.uint64), price=rng.uniform(0.5, 4.0, G),
        avail=rng.integers(40, 120, (n_zones, G)) * (1 if max_segments == 3 else 8), bw=bw)
    return prob.with_per_segment_tp(True).with_mixed_types(mixed)


@pytest.mark.parametrize("n_zones, mixed, max_segments", [(2, False, 3), (2, True, 3), (2, False, 2)])
def test_whole_units_guided_by_a_running_limit(torch_cuda, n_zones, mixed, max_segments):
    # the first units of the order are shared by workgroups, which divide the rounds of the lane space first and then
    # the innermost loop; the others have the degrees that a bound leaves only.  In the order of the availability at
    # creation, of which the second table leaves little.
    prob = _many_small_units(n_zones, mixed, max_segments)
    plan = _plan(prob)
    try:
        for avail in (prob.avail, prob.avail * 2 // 5):
            plan.set_avail(avail)
            orc = Oracle(prob.with_avail(avail))
            t, c, _, mask = orc.eval_batch(n_threads=THREADS)
            assert (mask == 0).sum() > 1000
            for objective in (MAX_THROUGHPUT, MIN_COST):
                val = (c if objective == MAX_THROUGHPUT else 1.0 / t)[mask == 0]
                for bound in (None, off_data(float(np.median(val)))):
                    check_result(plan.best_plan(objective=objective, bound=bound),
                                 orc.best(objective=objective, bound=bound, n_threads=THREADS), orc)
                    for k in (1, 64, 128):
                        check_topk(plan.topk(k, objective=objective, bound=bound),
                                   orc.topk(k, objective=objective, bound=bound, n_threads=THREADS), objective, orc, bound)
        assert plan.last_scan()[1] * 2 > 16384  # (two waves or more each, and none of them cut)
    finally:
        plan.destroy()
