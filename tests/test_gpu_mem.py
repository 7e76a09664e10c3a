"""GPU parity of cfp_dp_chain_mem + cfp_traceback against the CPU oracle:
optimum, status and plan must match bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_util import assert_mem_parity, need_gpu, run_mem, say
from workloads import configs, gen

pytestmark = pytest.mark.gpu
INF = gen.COST_INF


def mem_case(seed, B, N, K, E, lo, hi, mlo, mhi, M):
    rs = np.random.default_rng(seed)
    cost = rs.integers(lo, hi, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(lo, hi, size=(E, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = 0
    redge = (np.arange(N) % E).astype(np.int32)
    mem = rs.integers(mlo, mhi, size=(B, N, K)).astype(np.uint8)
    return cost, rtab, redge, mem


def test_config_full():
    need_gpu()
    say("config mem_llama_n288_k32")
    d = configs.make("mem_llama_n288_k32")
    assert_mem_parity(d["cost"], d["rtab"], d["redge"], d["mem"], d["M"], d["budget"], "mem config")


@pytest.mark.parametrize("N,K,M", [(1, 5, 10), (2, 3, 7), (13, 16, 64), (40, 32, 65), (70, 20, 130), (25, 32, 200),
                                   (90, 9, 300)])
def test_shapes(N, K, M):
    need_gpu()
    say("mem shape", N, K, M)
    cost, rtab, redge, mem = mem_case([N, K, M], 6, N, K, 12, 10_000, 1_000_000, 0, min(9, M), M)  # entries < M
    lo = mem.min(axis=2).sum(axis=1)
    hi = mem.max(axis=2).sum(axis=1)
    # budgets spanning infeasible, tight, middle, loose and the top bucket
    budget = np.array([max(int(lo[0]) - 1, 0), int(lo[1]), (int(lo[2]) + int(hi[2])) // 2, int(hi[3]), M - 1,
                       min(M - 1, int(lo[5]) + 3)], np.int32)
    budget = np.minimum(budget, M - 1)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"N={N} K={K} M={M}")


@pytest.mark.parametrize("K", [4, 32])
def test_heavy_ties(K):
    need_gpu()
    N, M = 30, 100
    cost, rtab, redge, mem = mem_case([7, K], 4, N, K, 3, 0, 3, 0, 3, M)
    budget = np.array([10, 20, 40, 99], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"ties K={K}")


def test_large_shifts_and_general_edges():
    need_gpu()
    rs = np.random.default_rng(11)
    B, N, K, E, M = 3, 50, 12, 5, 700
    cost = rs.integers(0, 10**6, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(0, 10**6, size=(E, K, K)).astype(np.int32)
    redge = rs.integers(0, E, size=N).astype(np.int32)
    mem = rs.integers(0, 17, size=(B, N, K)).astype(np.uint8)   # shifts up to the supported 16
    budget = np.array([699, 300, 150], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, "shift16")


def test_unavailable_and_statuses():
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, CFP_ST_INFEASIBLE
    cost, rtab, redge, mem = mem_case(12, 4, 20, 8, 2, 0, 100, 0, 5, 64)
    cost[0][cost[0] % 3 == 0] = INF
    cost[1, 5, :] = INF                         # infeasible
    mem[2, 3, 2] = 40                           # beyond the largest supported shift -> bad input
    budget = np.array([63, 63, 63, 2], np.int32)  # search 3: budget below the least memory plan
    opt, st, plan = run_mem(cost, rtab, redge, mem, 64, budget)
    assert st[1] == CFP_ST_INFEASIBLE and st[2] == CFP_ST_BADINPUT
    assert (plan[1] == -1).all() and (plan[2] == -1).all()
    good = [0, 3]
    assert_mem_parity(cost[good], rtab, redge, mem[good], 64, budget[good], "inf")


def test_budget_out_of_range_is_bad_input():
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT
    cost, rtab, redge, mem = mem_case(13, 2, 10, 4, 2, 0, 100, 0, 3, 32)
    opt, st, plan = run_mem(cost, rtab, redge, mem, 32, np.array([31, 32], np.int32))
    assert st[0] == 0 and st[1] == CFP_ST_BADINPUT


@pytest.mark.parametrize("bad", ["limit", "negative"])
def test_resharding_out_of_range_is_bad_input(bad):
    """The memory forward checks the range of R while packing it."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit
    cost, rtab, redge, mem = mem_case(14, 3, 30, 32, 3, 0, 100, 0, 4, 64)
    rtab[2, 31, 5] = cfp_r_limit(1, 32) if bad == "limit" else -1
    opt, st, plan = run_mem(cost, rtab, redge, mem, 64, np.array([63, 40, 20], np.int32))
    assert (st == CFP_ST_BADINPUT).all() and (plan == -1).all()


def test_periodic_layers():
    """Repeated layers (the same costs and memory every 12 blocks): many tied
    plans at every budget."""
    need_gpu()
    rs = np.random.default_rng(31)
    B, N, K, M = 4, 96, 32, 300
    cost = np.tile(rs.integers(0, 40, size=(B, 12, K)).astype(np.int32), (1, N // 12, 1))
    mem = np.tile(rs.integers(0, 5, size=(B, 12, K)).astype(np.uint8), (1, N // 12, 1))
    rtab = rs.integers(0, 40, size=(12, K, K)).astype(np.int32)
    redge = (np.arange(N) % 12).astype(np.int32)
    budget = np.array([60, 120, 200, 299], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, "periodic")


# The memory search takes any K up to 256 (padded to 32, 64, 96, 128, 192 or
# 256 states per workgroup) and any number of resharding tables (streamed from
# the cache): a segment of four blocks of three strategies has 81 plans
# (Sec. 5.5), and its memory is the sum over its blocks (Eq. M).

@pytest.mark.parametrize("N,K,E,M", [(40, 33, 12, 200), (40, 64, 12, 260), (30, 81, 12, 150), (25, 128, 5, 140),
                                     (20, 200, 3, 120), (16, 256, 12, 100), (50, 32, 20, 300), (30, 17, 40, 90)])
def test_wide_states_and_many_tables(N, K, E, M):
    """Budgets that bind (between the least-memory plan and the unconstrained plan's memory), ragged K."""
    need_gpu()
    from oracle import oracle as O
    from paper_2504_00598_amd import cfp_r_limit
    say("mem wide", N, K, E, M)
    rs = np.random.default_rng([15, N, K, E, M])
    B = 5
    cost = rs.integers(10_000, 1_000_000, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(10_000, min(1_000_000, cfp_r_limit(1, K)), size=(E, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = 0
    redge = rs.integers(0, E, size=N).astype(np.int32)
    mem = rs.integers(0, 9, size=(B, N, K)).astype(np.uint8)
    lo = mem.min(axis=2).sum(axis=1)
    _, free_plan, _ = O.chain(cost, rtab, redge)
    used = np.array([int(mem[b][np.arange(N), free_plan[b]].sum()) for b in range(B)])
    budget = np.minimum(M - 1, lo + (np.minimum(used, M - 1) - lo) * np.array([0, 1, 2, 3, 4]) // 5).astype(np.int32)
    budget[4] = M - 1
    g_opt, _ = assert_mem_parity(cost, rtab, redge, mem, M, budget, f"wide N={N} K={K} E={E} M={M}")
    assert (budget[:4] < used[:4]).all() or (lo == used).any()


def test_segment_plans_k81():
    """A memory search over model segments: 4 blocks x 3 strategies = 81 plans,
    plan cost = sum of its blocks' costs, plan memory = sum of its blocks'
    memory, resharding between segments from the boundary block pair only
    (the expanded 81 x 81 table of Sec. 4.2)."""
    need_gpu()
    from oracle import oracle as O
    say("mem segment plans K=81")
    rs = np.random.default_rng(16)
    B, N, M = 4, 48, 400
    P, S = 4, 3
    K = S ** P
    digits = np.array([[(t // S ** j) % S for j in range(P)] for t in range(K)])  # block strategies of plan t
    bc = rs.integers(10_000, 1_000_000, size=(B, N, P, S))
    bm = rs.integers(0, 3, size=(B, N, P, S))
    cost = np.zeros((B, N, K), np.int64)
    mem = np.zeros((B, N, K), np.int64)
    for j in range(P):
        cost += bc[:, :, j, :][:, :, digits[:, j]]
        mem += bm[:, :, j, :][:, :, digits[:, j]]
    cost = cost.astype(np.int32)
    mem = mem.astype(np.uint8)
    rbound = rs.integers(10_000, 10_000_000, size=(2, S, S)).astype(np.int32)
    rbound[:, np.arange(S), np.arange(S)] = 0
    last = digits[:, P - 1].astype(np.uint8)
    first = digits[:, 0].astype(np.uint8)
    rtab = O.expand_boundary(rbound, last, first)
    redge = np.ones(N, np.int32)
    redge[1] = 0
    lo = mem.min(axis=2).sum(axis=1)
    budget = np.minimum(M - 1, lo + np.array([0, 20, 60, 400])).astype(np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, "segment plans K=81")


def test_launch_rounds():
    """Many searches with many 64-bucket chunks each: the chunks of one launch
    must be resident together, so the searches run in several rounds."""
    need_gpu()
    say("mem launch rounds")
    rs = np.random.default_rng(17)
    B, N, K, M = 40, 20, 8, 4096
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(0, 1000, size=(3, K, K)).astype(np.int32)
    redge = (np.arange(N) % 3).astype(np.int32)
    mem = rs.integers(0, 17, size=(B, N, K)).astype(np.uint8)
    budget = rs.integers(0, M, size=B).astype(np.int32)
    budget[:4] = M - 1
    assert_mem_parity(cost, rtab, redge, mem, M, budget, "rounds")


def test_repeat_is_bit_identical():
    """The chunk pipeline gives the same bits on every run."""
    need_gpu()
    d = configs.make("mem_llama_n288_k32")
    first = run_mem(d["cost"], d["rtab"], d["redge"], d["mem"], d["M"], d["budget"])
    for _ in range(3):
        again = run_mem(d["cost"], d["rtab"], d["redge"], d["mem"], d["M"], d["budget"])
        for a, b in zip(first, again):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("N,K,M", [(30, 1, 33), (30, 16, 64), (25, 17, 50), (25, 47, 130), (20, 48, 129), (20, 49, 70),
                                   (15, 80, 90), (15, 97, 66), (12, 112, 130), (12, 128, 65)])
def test_padded_state_counts(N, K, M):
    """Every padded state count up to 128 (multiples of 16, odd ones with a last block of 16
    predecessors), bucket counts that are not whole 16-byte pieces."""
    need_gpu()
    say("mem padded states", N, K, M)
    cost, rtab, redge, mem = mem_case([80, N, K, M], 4, N, K, 5, 0, 1_000_000, 0, 9, M)
    cost[np.random.default_rng([81, K]).random(cost.shape) < 0.05] = INF
    budget = np.array([M - 1, M // 2, M // 3, 15], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"N={N} K={K} M={M}")


@pytest.mark.parametrize("N,K,mhi", [(150, 8, 1), (150, 8, 2), (90, 30, 17), (130, 5, 17), (20, 250, 17)])
def test_traceback_windows(N, K, mhi):
    """Windows of the plan recovery: no memory at all (64 rows each), small and the largest
    shifts (16), whole pieces and single buckets above 0, budgets that end in every place
    of a 16-byte piece."""
    need_gpu()
    say("mem traceback windows", N, K, mhi)
    M = 16 * N // 2 + 40 if K < 100 else 200
    M = min(M, 1500)
    cost, rtab, redge, mem = mem_case([82, N, K, mhi], 6, N, K, 3, 0, 1000, 0, mhi, M)
    budget = np.array([M - 1, M - 2, M - 9, M // 2, M // 2 + 16, M // 3], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"windows N={N} K={K} mhi={mhi}")


@pytest.mark.parametrize("head", [1, 3, 4])
def test_edge_map_with_a_head(head):
    """A head and a period of 61 entries: in the launch's arguments (64 entries together) or
    uploaded."""
    need_gpu()
    say("mem edge map", head)
    cost, rtab, redge, mem = mem_case([13, head], 3, 150, 12, 5, 10_000, 1_000_000, 0, 5, 70)
    redge = np.resize(np.random.default_rng(14).integers(0, 5, size=61), 150).astype(np.int32)
    redge[:head] = (redge[:head] + 1) % 5
    budget = np.array([69, 66, 63], np.int32)
    mem[:, 60:] = 0
    mem[:, :60] //= 4
    assert_mem_parity(cost, rtab, redge, mem, 70, budget, f"edge head {head}")


@pytest.mark.parametrize("K", [4, 17])
def test_many_searches_of_many_buckets(K):
    """More chunks than the device holds at once, and more steps than the rings can run
    ahead: searches wait for a round of their own, none for a chunk that cannot start."""
    need_gpu()
    N, M, B = 200, 1024, 64
    say("mem residency", K)
    cost, rtab, redge, mem = mem_case([83, K], B, N, K, 12, 10_000, 1_000_000, 0, 9, M)
    budget = np.array([M - 1 - (M // 32) * (i % 16) for i in range(B)], np.int32)
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"residency K={K}")
