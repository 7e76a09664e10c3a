"""GPU parity at the edges of the documented cost domain.

Costs may be any value in [0, CFP_COST_INF) (CFP_COST_INF marks an unavailable
strategy) and resharding entries any value in [0, cfp_r_limit).  These tests
draw costs uniformly from [0, 2^31 - 1) and put 0 and 2^31 - 2 into every
cost row, so that states far above a row's minimum (where the kernels cap
their normalised values) are reached by finite costs and not only by
unavailable strategies and padding.  Each shape is chosen to land on one
kernel family of the chain search (K <= 32 with tables in LDS, register-resident
K <= 64, chunk-parallel K <= 64, K <= 256 and K <= 512, state-split teams, split, split
with streamed tables, wide, the generic kernel for more tables than LDS holds), which
is checked, and the memory, frontier, scan and segment entry points get the same
treatment.  The bar is the oracle's answer
bit for bit: optimum, status and every plan entry (Sec. 4.4, Eq. T and Eq. M).
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import (assert_chain_parity, assert_form, assert_frontier_parity, assert_mem_parity,
                            assert_scan_parity, dev, need_gpu, oracle_threads, run_scan, say)
from workloads import gen

pytestmark = pytest.mark.gpu

INF = gen.COST_INF
TOP = INF - 1  # largest finite cost


def wide_costs(rs, B, N, K, inf_frac=0.0):
    """Uniform [0, 2^31 - 1) with a 0 and a 2^31 - 2 in every row (when K >= 2)."""
    cost = rs.integers(0, INF, size=(B, N, K), dtype=np.int64).astype(np.int32)
    if K >= 2:
        a = rs.integers(0, K, size=(B, N))
        b = (a + 1 + rs.integers(0, K - 1, size=(B, N))) % K
        np.put_along_axis(cost, a[..., None], 0, axis=2)
        np.put_along_axis(cost, b[..., None], TOP, axis=2)
    if inf_frac:
        cost[rs.random((B, N, K)) < inf_frac] = INF
    return cost


def wide_tables(rs, E, K, limit, zero_diag=False):
    rtab = rs.integers(0, limit, size=(E, K, K), dtype=np.int64).astype(np.int32)
    if zero_diag:
        rtab[:, np.arange(K), np.arange(K)] = 0
    return rtab


# (N, K, B, E, periodic edge map, form, kernel family the shape lands on)
CHAIN_CASES = [
    (50, 16, 3, 5, False, "NARROW", "tables in LDS, K<=16"),
    (60, 32, 3, 12, True, "NARROW", "tables in LDS, K<=32"),
    (40, 64, 3, 12, False, "ROWS", "register-resident K<=64, short chain"),
    (400, 64, 70, 12, True, "WAVE", "chunk-parallel K<=64, periodic tables (headerless)"),
    (300, 48, 20, 12, False, "WAVE", "chunk-parallel K<=64"),
    (50, 40, 3, 13, False, "WAVE", "one chunk K<=64, more than 12 tables"),
    (100, 100, 4, 12, False, "CHUNKS", "chunk-parallel K<=128"),
    (60, 100, 8, 17, False, "CHUNKS", "chunk-parallel K<=128, two chunks, more than 12 tables"),
    (200, 256, 9, 12, True, "CHUNKS", "chunk-parallel K<=256"),
    (100, 200, 3, 5, False, "CHUNKS", "chunk-parallel K<=256, ragged K"),
    (200, 512, 4, 12, True, "TEAMS", "chunk-parallel K<=512, state-split teams"),
    (150, 300, 3, 7, False, "TEAMS", "chunk-parallel K<=512, ragged K, state-split teams"),
    (360, 400, 12, 12, False, "CHUNKS", "chunk-parallel K<=512, several searches per workgroup"),
    (30, 100, 4, 12, False, "SPLIT", "split, tables in registers"),
    (130, 300, 3, 7, False, "SPLIT", "split, tables in registers, ragged K"),
    (30, 512, 2, 12, False, "SPLIT", "split K=512"),
    (30, 100, 8, 17, False, "SPLIT_STREAM", "split, streamed tables"),
    (200, 400, 12, 12, False, "SPLIT_STREAM", "split, streamed tables, K<=512"),
    (20, 100, 130, 3, False, "ROWS", "wide"),
    (15, 200, 66, 3, False, "ROWS", "wide K<=256"),
    (20, 300, 34, 3, False, "ROWS", "wide K<=512"),
    (50, 12, 3, 160, False, "ROWS", "generic K<=16"),
    (50, 30, 3, 40, False, "ROWS", "generic K<=32"),
]


@pytest.mark.parametrize("N,K,B,E,periodic,form,family", CHAIN_CASES, ids=[c[6] for c in CHAIN_CASES])
@pytest.mark.parametrize("rvals", ["full", "small"])
def test_chain_full_int32_costs(N, K, B, E, periodic, form, family, rvals):
    need_gpu()
    assert_form(form, N, K, B, E)
    from paper_2504_00598_amd import cfp_r_limit
    say("cost range chain", family, N, K, B, E, rvals)
    rs = np.random.default_rng([70, N, K, B, E, rvals == "full"])
    cost = wide_costs(rs, B, N, K, inf_frac=0.02)
    lim = cfp_r_limit(0, K) if rvals == "full" else 1000
    rtab = wide_tables(rs, E, K, lim, zero_diag=rvals == "small")
    redge = (np.arange(N) % E).astype(np.int32) if periodic else rs.integers(0, E, size=N).astype(np.int32)
    assert_chain_parity(cost, rtab, redge, f"{family} {rvals}")


@pytest.mark.parametrize("K", [16, 64, 256])
def test_chain_two_level_costs(K):
    """Every row holds only the two extremes 0 and 2^31 - 2 (and a few unavailable
    strategies): the normalised rows sit at 0 or at the cap almost everywhere,
    and the plan is decided by resharding entries alone."""
    need_gpu()
    say("two-level costs", K)
    rs = np.random.default_rng([71, K])
    B, N = 4, 150
    cost = np.where(rs.random((B, N, K)) < 0.5, 0, TOP).astype(np.int32)
    cost[rs.random((B, N, K)) < 0.03] = INF
    cost[:, :, 0] = np.where(cost[:, :, 0] == INF, TOP, cost[:, :, 0])  # keep every block feasible
    rtab = rs.integers(0, 50, size=(12, K, K)).astype(np.int32)
    redge = (np.arange(N) % 12).astype(np.int32)
    assert_chain_parity(cost, rtab, redge, f"two-level K={K}")


def test_scan_full_int32_costs():
    """The scan keeps products relative to their minimum in 32 bits, so it
    documents that the available costs of one block must lie within 2^30 of
    each other.  Inside that band, with costs up to 2^31 - 2, it is exact;
    a block that spreads wider is reported as bad input, never answered
    wrongly."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit
    say("cost range scan")
    rs = np.random.default_rng(72)
    B, N, K = 3, 70, 64
    lo = INF - 2**30
    cost = rs.integers(lo, INF - 1, size=(B, N, K), dtype=np.int64).astype(np.int32)
    cost[:, :, 0] = lo
    cost[:, :, 1] = TOP
    rtab = wide_tables(rs, 12, K, cfp_r_limit(2, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    assert_scan_parity(cost, rtab, redge, "scan band")
    wide = cost.copy()
    wide[1, 33, 5] = 0  # spread of 2^31 - 2 in one block of search 1
    opt, st, plan = run_scan(wide, rtab, redge)
    assert st[1] == CFP_ST_BADINPUT and opt[1] == np.iinfo(np.int64).max and (plan[1] == -1).all()
    o_opt, o_plan, o_st = O.chain(wide, rtab, redge, nthreads=oracle_threads())
    np.testing.assert_array_equal(opt[[0, 2]], o_opt[[0, 2]])
    np.testing.assert_array_equal(plan[[0, 2]], o_plan[[0, 2]])


def test_mem_two_block_large_gap():
    """Two blocks.  Block 0: strategy 0 costs 0 with one bucket, strategy 1 costs
    2^31 - 2 with none.  Block 1: every strategy costs 5 with one bucket.  At
    budget 1 only the dear first strategy fits, so the optimum is 2^31 + 3; at
    budget 2 it is 5.  The least cost of a column can therefore sit 2^31 above
    the least cost of a column with fewer buckets."""
    need_gpu()
    say("memory two-block gap")
    K = 4
    cost = np.full((3, 2, K), 5, np.int32)
    cost[:, 0, :] = INF
    cost[:, 0, 0] = 0
    cost[:, 0, 1] = TOP
    mem = np.ones((3, 2, K), np.uint8)
    mem[:, 0, 1] = 0
    rtab = np.zeros((1, K, K), np.int32)
    redge = np.zeros(2, np.int32)
    g_opt, _ = assert_mem_parity(cost, rtab, redge, mem, 4, [1, 2, 3], "two-block gap")
    assert g_opt.tolist() == [2**31 + 3, 5, 5]
    assert_frontier_parity(cost, rtab, redge, mem, 4, "two-block gap frontier")


@pytest.mark.parametrize("K,M", [(16, 200), (32, 300), (81, 150), (256, 100)])
def test_mem_full_int32_costs(K, M):
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    say("cost range memory", K, M)
    rs = np.random.default_rng([73, K, M])
    B, N = 6, 60 if K <= 32 else 25
    cost = wide_costs(rs, B, N, K, inf_frac=0.02)
    rtab = wide_tables(rs, 12, K, cfp_r_limit(1, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    mem = rs.integers(0, 9, size=(B, N, K)).astype(np.uint8)
    lo = mem.min(axis=2).sum(axis=1)
    budget = np.minimum(M - 1, lo + rs.integers(0, 3 * N, size=B)).astype(np.int32)
    budget[0] = M - 1
    assert_mem_parity(cost, rtab, redge, mem, M, budget, f"memory K={K}")
    assert_frontier_parity(cost, rtab, redge, mem, M, f"frontier K={K}")


@pytest.mark.parametrize("B,N,form", [(5, 80, "SEG_CLASS"), (5, 1500, "SEG_CHUNKS"), (800, 40, "SEG_ROWS")])
def test_segments_full_int32_costs(B, N, form):
    need_gpu()
    import torch
    from paper_2504_00598_amd import _lib as L
    from paper_2504_00598_amd import cfp_r_limit, search
    from oracle import oracle as OR
    say("cost range segments", form)
    rs = np.random.default_rng(74)
    K, Lc, Fc, E = 81, 3, 3, 2
    assert L.cfp_segment_form(N, K, B, E, Lc, Fc) == getattr(L, "CFP_FORM_" + form)
    cost = wide_costs(rs, B, N, K, inf_frac=0.02)
    rbound = rs.integers(0, cfp_r_limit(3, K), size=(E, Lc, Fc), dtype=np.int64).astype(np.int32)
    last = (np.arange(K) // 27).astype(np.uint8)
    first = (np.arange(K) % 3).astype(np.uint8)
    redge = rs.integers(0, E, size=N).astype(np.int32)
    r = search.dp_segments(dev(cost), dev(rbound), dev(last), dev(first), redge)
    torch.cuda.synchronize()
    o_opt, o_plan, o_st = OR.segments(cost, rbound, last, first, redge, nthreads=oracle_threads())
    np.testing.assert_array_equal(r.status.cpu().numpy(), o_st)
    np.testing.assert_array_equal(r.opt.cpu().numpy(), o_opt)
    np.testing.assert_array_equal(r.plan.cpu().numpy(), o_plan)
