"""What a plan allocates after its creation: larger selection buffers, beside work on other streams
and where there is no memory for them, and what kept minima take."""
import os
import subprocess
import sys

import numpy as np
import pytest

from oracle.oracle import MAX_THROUGHPUT, MIN_COST, Oracle
from paper_2504_17096_amd import workloads as W
from tests.helpers import make_problem

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def crowded_problem():
    """110 592 plans, all of them valid, in nine pieces: no 128 waves that could name a key each, so the first
    pass of a query for the 128 best keeps them all, and the 64 Ki entries of a new plan do not hold them."""
    rng = np.random.default_rng(17)
    G, Z, mb, tp = 4, 16, (1, 2, 3, 4, 6, 8, 12, 24), (1, 2, 4)
    dp = (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 15, 16, 18, 20, 21, 24, 28, 30, 35, 36, 40, 42)
    bw = rng.uniform(0.5e9, 2e9, (Z, Z))
    np.fill_diagonal(bw, rng.uniform(0.8e10, 1.2e10, Z))
    return make_problem(
        n_layers=6, n_types=G, n_zones=Z, mb_list=mb, tp_list=tp, dp_list=dp, pp_list=[1, 2, 3],
        global_batch=24 * 5040, max_segments=1, t_fwd=rng.uniform(0.5e-3, 3e-3, (G, len(mb), 3, 1)),
        t_bwd=rng.uniform(1e-3, 5e-3, (G, len(mb), 3, 1)), t_upd=rng.uniform(1e-4, 3e-4, (G, 3, 1)),
        p2p=rng.integers(1_000_000, 9_000_000, len(mb)).astype(np.uint64), cap=1 << 40,
        price=rng.uniform(0.5, 4.0, G), avail=100_000, bw=bw)


def check_top(got, want):
    assert [r.index for r in got] == [w.index for w in want]
    for r, w in zip(got, want):
        assert r.iter_time_s == pytest.approx(w.iter_time, rel=1e-9)
        assert r.cost_per_iter == pytest.approx(w.cost, rel=1e-9)


@pytest.mark.parametrize("objective", [MAX_THROUGHPUT, MIN_COST])
def test_buffers_grow_beside_work_on_other_streams(torch_cuda, objective):
    from paper_2504_17096_amd.binding import Plan
    torch = torch_cuda
    plan, orc = Plan(crowded_problem()), Oracle(crowded_problem())
    try:
        want = orc.topk(128, objective, n_threads=4)
        query = torch.cuda.Stream()

        def beside(cycles, k):
            """The k best plans, and whether they came while the other stream was at work."""
            done = torch.cuda.Event()
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                torch.cuda._sleep(cycles)
                done.record()
            got = plan.topk(k, objective=objective, stream=query.cuda_stream)
            return got, not done.query()

        for _ in range(8):  # a stream that does not share its hardware queue with the query's
            side = torch.cuda.Stream()
            got, at_work = beside(200_000_000, 4)
            check_top(got, want[:4])
            if at_work:
                break
        assert at_work and plan.last_counts()[0] <= 1 << 16
        got, at_work = beside(1_000_000_000, 128)
        assert at_work, "the query waited for the other stream"
        check_top(got, want)
        assert plan.last_counts()[0] > 1 << 16  # (they have grown)
    finally:
        plan.destroy()


def test_minima_kept_from_within_a_capture_on(torch_cuda):
    from paper_2504_17096_amd.binding import Plan
    torch = torch_cuda
    prob = W.config2()
    plan, other = Plan(prob), Plan(prob)
    try:
        n = other.num_candidates()
        t = torch.zeros(n, dtype=torch.float32, device="cuda:0")
        side = torch.cuda.Stream()
        other.eval_batch(0, n, d_time=t)
        torch.cuda.synchronize()
        want = t.cpu().numpy()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            plan.set_incremental(True)
            other.eval_batch(0, n, d_time=t, stream=side.cuda_stream)
        assert plan.best_plan().index == plan.best_plan().index == Oracle(prob).best().index
        assert plan.last_scan()[0] == 0  # the second call found the first one's minima
        for _ in range(3):
            t.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(t.cpu().numpy(), want)
    finally:
        plan.destroy()
        other.destroy()


def refused_queries():
    """(in a process of its own, see below)"""
    import ctypes
    from tests.abi_example import build
    refusal = ctypes.CDLL(build.build_refusal(force=False), ctypes.RTLD_GLOBAL)
    refusal.refuse_from.argtypes = [ctypes.c_size_t]
    from paper_2504_17096_amd.binding import SAILOR_ENOMEM, Plan, SailorError
    prob = crowded_problem()
    orc, plan = Oracle(prob), Plan(prob)
    refusal.refuse_from(4 << 20)  # the first buffers have 2 MiB, the larger ones 106
    for objective in (MAX_THROUGHPUT, MIN_COST):
        for repeat in range(2):
            before = refusal.times_refused()
            check_top(plan.topk(128, objective=objective), orc.topk(128, objective, n_threads=4))
            assert refusal.times_refused() > before and plan.last_counts()[0] <= 1 << 16
        assert plan.best_plan(objective=objective).index == orc.best(objective).index
    refusal.refuse_from((1 << 64) - 1)  # there is memory again
    check_top(plan.topk(128), orc.topk(128, n_threads=4))
    assert plan.last_counts()[0] > 1 << 16
    plan.destroy()
    plan = Plan(prob)
    refusal.refuse_from(50_000)  # 9 pieces of 6 400 bytes: nothing is kept without memory for them, and no error is left
    try:
        plan.set_incremental(True)
        raise AssertionError("not refused")
    except SailorError as e:
        assert e.status == SAILOR_ENOMEM
    assert plan.best_plan().index == plan.best_plan().index == orc.best().index
    refusal.refuse_from((1 << 64) - 1)
    plan.set_incremental(True)
    assert plan.best_plan().index == plan.best_plan().index == orc.best().index and plan.last_scan()[0] == 0
    plan.destroy()
    print("refused_queries: OK")


def test_queries_go_on_without_memory_for_larger_buffers(torch_cuda):
    run = subprocess.run([sys.executable, "-c", "from tests.test_gpu_scratch import refused_queries; refused_queries()"],
                         cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "refused_queries: OK" in run.stdout
