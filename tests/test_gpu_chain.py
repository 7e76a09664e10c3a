"""GPU parity of cfp_dp_chain + cfp_traceback against the CPU oracle:
optimum, status and plan must match bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import assert_chain_parity, assert_form, dev, need_gpu, oracle_threads, run_chain, say
from workloads import configs, gen

pytestmark = pytest.mark.gpu

INF = gen.COST_INF


def rand_case(seed, B, N, K, E, lo, hi, rlo=None, rhi=None, inf_frac=0.0):
    rs = np.random.default_rng(seed)
    cost = rs.integers(lo, hi, size=(B, N, K)).astype(np.int32)
    if inf_frac:
        cost[rs.random((B, N, K)) < inf_frac] = INF
    rtab = rs.integers(lo if rlo is None else rlo, hi if rhi is None else rhi, size=(E, K, K)).astype(np.int32)
    redge = rs.integers(0, E, size=N).astype(np.int32)
    return cost, rtab, redge


@pytest.mark.parametrize("cfg", ["chain_gpt_n24_k16", "chain_gpt_n1152_k64", "chain_wide_n512_k256"])
def test_configs_full(cfg):
    need_gpu()
    say("config", cfg)
    d = configs.make(cfg)
    assert_chain_parity(d["cost"], d["rtab"], d["redge"], cfg)


SHAPES = [(1, 1), (1, 5), (2, 1), (3, 2), (7, 3), (65, 16), (130, 17), (129, 31), (64, 32), (70, 33),
          (200, 64), (66, 65), (131, 100), (90, 128), (40, 129), (67, 200), (33, 256), (20, 257), (9, 300),
          (12, 512)]


@pytest.mark.parametrize("N,K", SHAPES)
def test_shapes_realistic_values(N, K):
    need_gpu()
    say("shape", N, K)
    from paper_2504_00598_amd import cfp_r_limit
    rhi = min(10_000_000, cfp_r_limit(0, K))  # resharding values within the documented exact range
    cost, rtab, redge = rand_case([1, N, K], 3, N, K, 5, 10_000, 10_000_000, rlo=10_000, rhi=rhi)
    assert_chain_parity(cost, rtab, redge, f"N={N} K={K}")


@pytest.mark.parametrize("N,K", SHAPES)
def test_shapes_heavy_ties(N, K):
    need_gpu()
    say("ties", N, K)
    cost, rtab, redge = rand_case([2, N, K], 2, N, K, 3, 0, 3)
    assert_chain_parity(cost, rtab, redge, f"ties N={N} K={K}")


@pytest.mark.parametrize("K", [16, 64, 200, 512])
def test_largest_allowed_resharding(K):
    """R entries at cfp_r_limit - 1 and costs near 2^31: still exact."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    lim = cfp_r_limit(0, K)
    rs = np.random.default_rng(K)
    N = 50
    cost = rs.integers(2**31 - 10**6, 2**31 - 1, size=(2, N, K)).astype(np.int32)
    rtab = rs.integers(lim - 1000, lim, size=(4, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = rs.integers(0, 3, size=(4, K))
    redge = rs.integers(0, 4, size=N).astype(np.int32)
    assert_chain_parity(cost, rtab, redge, f"max R K={K}")


@pytest.mark.parametrize("K", [3, 64, 256])
def test_unavailable_strategies(K):
    need_gpu()
    cost, rtab, redge = rand_case([3, K], 4, 40, K, 3, 0, 100, inf_frac=0.3)
    cost[1, 7, :] = INF        # search 1: every strategy of block 7 unavailable -> infeasible
    cost[2, 0, :] = INF        # search 2: block 0 unavailable -> infeasible
    cost[3, :, 1:] = INF       # search 3: only strategy 0 is left anywhere
    cost[3, :, 0] = 5
    g_opt, g_plan = assert_chain_parity(cost, rtab, redge, f"inf K={K}")
    assert (g_plan[1] == -1).all() and (g_plan[2] == -1).all()
    assert (g_plan[3] == 0).all()


def test_badinput_statuses():
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit
    cost, rtab, redge = rand_case(4, 3, 20, 16, 2, 0, 100)
    cost[1, 3, 4] = -5
    opt, st, plan = run_chain(cost, rtab, redge)
    assert st.tolist() == [0, CFP_ST_BADINPUT, 0]
    assert opt[1] == np.iinfo(np.int64).max and (plan[1] == -1).all()
    rtab2 = rtab.copy()
    rtab2[1, 2, 3] = cfp_r_limit(0, 16)
    opt, st, plan = run_chain(cost, rtab2, redge)
    assert (st == CFP_ST_BADINPUT).all() and (plan == -1).all()


def test_repeat_is_bit_identical():
    need_gpu()
    d = configs.make("chain_gpt_n1152_k64", batch=32)
    first = run_chain(d["cost"], d["rtab"], d["redge"])
    for _ in range(3):
        again = run_chain(d["cost"], d["rtab"], d["redge"])
        for a, b in zip(first, again):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("K", [16, 64, 100, 256])
def test_periodic_layers(K):
    """Every layer of 12 blocks repeats the same costs (profiles of one
    distinct segment reused for every instance, Sec. 4.1): a search space
    full of equal-cost plans, so the lowest-index rule decides the plan."""
    need_gpu()
    rs = np.random.default_rng(30 + K)
    B, N = 4, 240
    layer = rs.integers(0, 30, size=(B, 12, K)).astype(np.int32)
    cost = np.tile(layer, (1, N // 12, 1))
    rtab = rs.integers(0, 30, size=(12, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = 0
    redge = (np.arange(N) % 12).astype(np.int32)
    say("periodic layers", K)
    assert_chain_parity(cost, rtab, redge, f"periodic K={K}")


# The traceback follows the argmin table in one launch from LDS when a search's
# table fits there (about 150 KiB: N K bytes, 2 N K for K > 256) and in three
# launches from memory otherwise; shapes on both sides of that boundary, with
# ties so that many chains of the traceback merge.
@pytest.mark.parametrize("N,K,B", [(512, 256, 2), (1152, 64, 2), (129, 512, 1), (300, 129, 2),
                                   (600, 256, 2), (2600, 64, 2), (160, 512, 1), (300, 257, 1)])
def test_traceback_lds_and_memory_paths(N, K, B):
    need_gpu()
    say("traceback path", N, K, B)
    cost, rtab, redge = rand_case([7, N, K], B, N, K, 4, 0, 50)
    assert_chain_parity(cost, rtab, redge, f"traceback N={N} K={K}")


# The chunk-parallel paths check the range of R while packing it (the other
# paths in a separate pass): an entry at cfp_r_limit or below 0 marks every
# search of the call as bad input.
@pytest.mark.parametrize("N,K,B,bad,form", [
    (400, 64, 70, "limit", "WAVE"), (400, 64, 70, "negative", "WAVE"), (200, 256, 9, "limit", "CHUNKS"),
    (200, 256, 9, "negative", "CHUNKS"), (20, 16, 3, "limit", "NARROW"), (200, 300, 3, "negative", "TEAMS"),
    (30, 100, 3, "limit", "SPLIT"), (30, 100, 70, "negative", "SPLIT_STREAM"), (30, 100, 130, "limit", "ROWS"),
    (30, 64, 3, "negative", "ROWS")])
def test_resharding_range_checked_on_every_path(N, K, B, bad, form):
    need_gpu()
    assert_form(form, N, K, B, 12)
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit
    say("R range", N, K, B, bad)
    cost, rtab, redge = rand_case([48, N, K], B, N, K, 12, 0, 1000)
    redge = (np.arange(N) % 12).astype(np.int32)
    opt, st, plan = run_chain(cost, rtab, redge)
    assert (st == 0).all()
    rtab[7, K - 1, K // 2] = cfp_r_limit(0, K) if bad == "limit" else -1
    opt, st, plan = run_chain(cost, rtab, redge)
    assert (st == CFP_ST_BADINPUT).all() and (opt == np.iinfo(np.int64).max).all() and (plan == -1).all()


# Chains of K > 64 too short to be cut into chunks (up to 32 rows of K <= 256, and those of
# K > 256 that take less time row after row) run on three kernels.  Two split a search over
# several workgroups that must all fit the device's 256 compute units: K_P^2 / 4096 of them
# with the tables in registers (K_P the padded K, at most 12 tables), or K_P / 64 that stream
# the tables.  The third is the wide kernel, one workgroup per search.

@pytest.mark.parametrize("N,K,B,E", [(30, 100, 129, 12), (32, 65, 300, 12), (32, 128, 140, 12), (1, 100, 200, 3),
                                     (31, 200, 65, 12), (15, 256, 300, 12), (2, 130, 90, 17), (40, 300, 33, 12),
                                     (127, 512, 40, 12), (9, 257, 50, 17)])
def test_wide_path_batches(N, K, B, E):
    """Batches too large for the split kernels: the wide kernel."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("ROWS", N, K, B, E)
    say("wide path", N, K, B)
    rhi = min(10_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([3, K, B], B, N, K, E, 10_000, 10_000_000, rlo=10_000, rhi=rhi)
    assert_chain_parity(cost, rtab, redge, f"wide N={N} K={K} B={B}")


@pytest.mark.parametrize("N,K,B,E", [(32, 65, 65, 12), (32, 128, 128, 12), (20, 100, 2, 17), (2, 100, 5, 13),
                                     (30, 200, 17, 12), (32, 256, 64, 12), (31, 150, 2, 17), (40, 300, 5, 12),
                                     (143, 512, 8, 12), (351, 400, 32, 12), (60, 257, 1, 17)])
def test_split_path_streamed_tables(N, K, B, E):
    """Batches or tables too many for the registers: slices of the tables streamed."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("SPLIT_STREAM", N, K, B, E)
    say("split path, streamed", N, K, B, E)
    rhi = min(1_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([6, N, K, B], B, N, K, E, 10_000, 1_000_000, rlo=10_000, rhi=rhi, inf_frac=0.02)
    assert_chain_parity(cost, rtab, redge, f"split, streamed N={N} K={K} B={B} E={E}")


@pytest.mark.parametrize("N,K,B", [(32, 65, 4), (30, 128, 64), (2, 100, 3), (31, 256, 16), (17, 130, 5), (120, 257, 4),
                                   (127, 512, 4), (143, 400, 3)])
def test_split_path_long_chains(N, K, B):
    """Few chains spread over many workgroups (B * P = 256 at the largest), of up to the
    most rows that go row after row."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("SPLIT", N, K, B, 12)
    say("split path", N, K, B)
    rhi = min(1_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([5, N, K, B], B, N, K, 12, 10_000, 1_000_000, rlo=10_000, rhi=rhi)
    assert_chain_parity(cost, rtab, redge, f"split N={N} K={K} B={B}")


def test_long_chain_workload():
    """The 4096-block K=512 workload of the scan through the chain search (64
    chunks of 64 rows)."""
    need_gpu()
    assert_form("TEAMS", 4096, 512, 4, 12)
    say("config scan_n4096_k512 through cfp_dp_chain")
    d = configs.make("scan_n4096_k512")
    assert_chain_parity(d["cost"], d["rtab"], d["redge"], "long chain K=512")


# 32 < K <= 64 on long chains (at least 8 blocks of 12 rows), and with more than 12 tables on
# any, runs chunk-parallel: the chains are cut into chunks that are searched concurrently
# from arbitrary start rows and then repaired until their rows meet the speculative ones; a
# chain whose rows never meet is finished sequentially.  Whatever happens inside, the
# answer must be the oracle's.

def _no_switch_tables(rs, E, K, lim):
    """Resharding so dear that no plan ever switches strategy: the rows of two runs
    started from different rows never become parallel, so no chunk's fix-up meets
    its speculative run."""
    rtab = rs.integers(lim - 1000, lim, size=(E, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = 0
    return rtab


@pytest.mark.parametrize("K,B", [(64, 3), (64, 70), (40, 9)])
def test_chunked_rows_never_meet(K, B):
    """Every chunk misses its checkpoints: the final pass reruns the chains."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([40, K, B])
    N = 600
    cost = rs.integers(0, 50, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 12, K, cfp_r_limit(0, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    say("chunked, no convergence", K, B)
    assert_chain_parity(cost, rtab, redge, f"never meet K={K} B={B}")


@pytest.mark.parametrize("seed", range(4))
def test_chunked_some_chunks_meet(seed):
    """A zero table (any row maps to a parallel one) placed on a few edges: chunks that
    contain one meet their speculative run, the others do not, in a seeded pattern."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([41, seed])
    K, B, N = 64, 68, 900
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    resets = rs.choice(np.arange(1, N), size=int(rs.integers(1, 6)), replace=False)
    redge[resets] = 2
    say("chunked, partial convergence", seed, sorted(resets.tolist()))
    assert_chain_parity(cost, rtab, redge, f"partial seed={seed}")


@pytest.mark.parametrize("N,K,B", [(96, 64, 256), (100, 64, 255), (1000, 33, 67), (777, 48, 130), (1152, 64, 1),
                                   (2000, 64, 8), (481, 63, 512)])
def test_chunked_shapes(N, K, B):
    """Ragged batches (searches beyond the last full group of a workgroup), ragged last
    blocks, K below 64 and chunk counts from 2 to 64."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("WAVE", N, K, B, 12)
    rhi = min(10_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([42, N, K, B], B, N, K, 12, 10_000, 10_000_000, rlo=10_000, rhi=rhi)
    if N % 2:
        redge = (np.arange(N) % 12).astype(np.int32)  # the periodic (register-set) table selection
    say("chunked shape", N, K, B)
    assert_chain_parity(cost, rtab, redge, f"chunked N={N} K={K} B={B}")


def test_chunked_ties_and_statuses():
    """Tie-heavy values, unavailable strategies and bad inputs on the chunked path."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT
    cost, rtab, redge = rand_case([43], 70, 400, 64, 5, 0, 3, inf_frac=0.1)
    cost[5, 250, :] = INF   # infeasible search, in a late chunk
    assert_chain_parity(cost, rtab, redge, "chunked ties")
    cost[9, 100, 3] = -7    # a negative cost is rejected by the library (the oracle has no such check)
    opt, st, plan = run_chain(cost, rtab, redge)
    assert st[9] == CFP_ST_BADINPUT and opt[9] == np.iinfo(np.int64).max and (plan[9] == -1).all()
    assert st[5] != 0 and (st[np.r_[0:5, 6:9, 10:70]] == 0).all()


# 128 < K <= 256 on chains of more than 32 blocks runs chunk-parallel as well, with two or
# four chains per workgroup sharing each streamed table word.  Same requirement: the
# oracle's answer whatever the rows do.

@pytest.mark.parametrize("N,K,B", [(36, 256, 1), (33, 129, 2), (100, 200, 3), (513, 256, 64), (1000, 255, 5),
                                   (257, 160, 64), (64, 256, 129), (81, 256, 2)])
def test_chunked_wide_shapes(N, K, B):
    """Ragged batches (an odd last search), ragged last chunks, K below 256, one-row chunks."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("CHUNKS", N, K, B, 12)
    rhi = min(10_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([44, N, K, B], B, N, K, 12, 10_000, 10_000_000, rlo=10_000, rhi=rhi)
    if N % 2:
        redge = (np.arange(N) % 12).astype(np.int32)
    say("chunked wide shape", N, K, B)
    assert_chain_parity(cost, rtab, redge, f"chunked wide N={N} K={K} B={B}")


@pytest.mark.parametrize("K,B", [(256, 3), (200, 8)])
def test_chunked_wide_rows_never_meet(K, B):
    """Every chunk misses its checkpoints: the final pass reruns the chains."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([45, K, B])
    N = 300
    cost = rs.integers(0, 50, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 12, K, cfp_r_limit(0, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    say("chunked wide, no convergence", K, B)
    assert_chain_parity(cost, rtab, redge, f"wide never meet K={K} B={B}")


@pytest.mark.parametrize("seed", range(3))
def test_chunked_wide_some_chunks_meet(seed):
    """Zero tables on a few edges make some chunks meet and others not, in a seeded pattern."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([46, seed])
    K, B, N = 256, 6, 600
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    resets = rs.choice(np.arange(1, N), size=int(rs.integers(1, 6)), replace=False)
    redge[resets] = 2
    say("chunked wide, partial convergence", seed, sorted(resets.tolist()))
    assert_chain_parity(cost, rtab, redge, f"wide partial seed={seed}")


def test_chunked_wide_ties_and_statuses():
    """Tie-heavy values, unavailable strategies, an infeasible search and a negative cost."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT
    cost, rtab, redge = rand_case([47], 9, 200, 256, 5, 0, 3, inf_frac=0.1)
    cost[4, 150, :] = INF   # infeasible search, in a late chunk
    assert_chain_parity(cost, rtab, redge, "chunked wide ties")
    cost[7, 60, 3] = -7     # a negative cost is rejected by the library
    opt, st, plan = run_chain(cost, rtab, redge)
    assert st[7] == CFP_ST_BADINPUT and opt[7] == np.iinfo(np.int64).max and (plan[7] == -1).all()
    assert st[4] != 0 and st[6] == 0 and st[8] == 0 and (st[np.r_[0:4, 5:7]] == 0).all()


def test_header_uploads_back_to_back():
    """Forty calls enqueued without a synchronisation, each with its own edge
    map and workspace: more calls than the library's ring of pinned upload
    slots, so slots are reused while earlier copies may still be queued."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import search
    say("header uploads back to back")
    rs = np.random.default_rng(61)
    B, N, K, E = 2, 40, 16, 4
    rtab = rs.integers(0, 50, size=(E, K, K)).astype(np.int32)
    cases, results = [], []
    for c in range(40):
        cost = rs.integers(0, 50, size=(B, N, K)).astype(np.int32)
        redge = rs.integers(0, E, size=N).astype(np.int32)
        cases.append((cost, redge))
        results.append(search.dp_chain(dev(cost), dev(rtab), redge))
    torch.cuda.synchronize()
    for c, ((cost, redge), r) in enumerate(zip(cases, results)):
        o_opt, o_plan, o_st = O.chain(cost, rtab, redge)
        np.testing.assert_array_equal(r.opt.cpu().numpy(), o_opt, err_msg=f"opt call {c}")
        np.testing.assert_array_equal(r.plan.cpu().numpy(), o_plan, err_msg=f"plan call {c}")


def test_range_flag_does_not_leak_between_calls():
    """The chunk-parallel K=64 path with a periodic edge map does not upload the
    workspace header and flags an out-of-range R by call number: a workspace
    reused after a call with bad R, or after a call on another path, gives
    clean statuses."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit, search
    say("range flag across calls")
    rs = np.random.default_rng(62)
    B, N, K = 70, 400, 64
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(0, 1000, size=(12, K, K)).astype(np.int32)
    periodic = (np.arange(N) % 12).astype(np.int32)
    bad = rtab.copy()
    bad[3, 5, 7] = cfp_r_limit(0, K)
    r = search.dp_chain(dev(cost), dev(bad), periodic)
    torch.cuda.synchronize()
    assert (r.status.cpu().numpy() == CFP_ST_BADINPUT).all()
    ws = r.ws
    o_opt, o_plan, o_st = O.chain(cost, rtab, periodic, nthreads=oracle_threads())
    r2 = search.dp_chain(dev(cost), dev(rtab), periodic, ws=ws)  # same workspace, good R
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r2.status.cpu().numpy(), o_st)
    np.testing.assert_array_equal(r2.opt.cpu().numpy(), o_opt)
    np.testing.assert_array_equal(r2.plan.cpu().numpy(), o_plan)
    # a non-periodic edge map (another path, header uploaded) with bad R, then periodic again
    other = rs.integers(0, 12, size=N).astype(np.int32)
    r3 = search.dp_chain(dev(cost), dev(bad), other, ws=ws)
    torch.cuda.synchronize()
    assert (r3.status.cpu().numpy() == CFP_ST_BADINPUT).all()
    r4 = search.dp_chain(dev(cost), dev(rtab), periodic, ws=ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(r4.opt.cpu().numpy(), o_opt)
    np.testing.assert_array_equal(r4.plan.cpu().numpy(), o_plan)


def test_range_flag_ignores_stale_workspace_bytes():
    """The headerless K=64 path keeps its range flag in a workspace word that no
    upload clears.  Fresh workspaces whose flag word holds small integers,
    all-ones, or other leftovers (a freed plan row, an earlier cost) must still
    give a clean search."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import _lib as L, search
    say("range flag with stale workspace bytes")
    rs = np.random.default_rng(63)
    B, N, K = 70, 400, 64
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = rs.integers(0, 1000, size=(12, K, K)).astype(np.int32)
    periodic = (np.arange(N) % 12).astype(np.int32)
    o_opt, o_plan, o_st = O.chain(cost, rtab, periodic, nthreads=oracle_threads())
    d = L.Desc(dev(cost), dev(rtab), periodic)
    nbytes = L.cfp_workspace_bytes(d, L.CFP_V_CHAIN)
    words = list(range(0, 65)) + [-1, 2**31 - 1, 2**32, 2**63 - 1, -(2**63), int(rs.integers(0, 2**62))]
    for v in words:
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ws[:64].view(torch.int64)[:] = v   # every 8-byte word of the first 64 bytes, the flag word among them
        r = search.dp_chain(d.cost, d.rtab, periodic, ws=ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(r.status.cpu().numpy(), o_st, err_msg=f"status, stale word {v}")
        np.testing.assert_array_equal(r.opt.cpu().numpy(), o_opt, err_msg=f"opt, stale word {v}")
        np.testing.assert_array_equal(r.plan.cpu().numpy(), o_plan, err_msg=f"plan, stale word {v}")


# 256 < K <= 512 runs chunk-parallel with chunks of at least 48 rows (runs take tens of
# rows to become parallel at this width): batches of at most 8 searches from 144 blocks on
# in state-split teams (four workgroups per chunk, rows exchanged every step), larger ones
# with two or four searches per workgroup from 352 blocks on, or 128 if no split kernel
# takes them.  The final pass reruns, whole, each chunk whose start row was not the true one.

@pytest.mark.parametrize("N,K,B", [(144, 512, 1), (300, 400, 5), (1000, 512, 3), (640, 300, 8), (145, 257, 2),
                                   (4096, 512, 1), (700, 512, 12), (352, 300, 9), (1200, 511, 7), (130, 260, 50)])
def test_chunked_k512_shapes(N, K, B):
    """Three chunks of 48 rows, ragged K and batches, ragged last chunks, 64 chunks;
    teams of one and two groups of searches, and several searches per workgroup."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("TEAMS" if B <= 8 else "CHUNKS", N, K, B, 12)
    rhi = min(1_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([48, N, K, B], B, N, K, 12, 10_000, 1_000_000, rlo=10_000, rhi=rhi)
    if N % 2 == 0:
        redge = (np.arange(N) % 12).astype(np.int32)
    say("chunked K>256 shape", N, K, B)
    assert_chain_parity(cost, rtab, redge, f"chunked K>256 N={N} K={K} B={B}")


@pytest.mark.parametrize("N,K,B", [(1105, 512, 1), (1106, 400, 5), (1107, 512, 3)])
def test_chunked_k512_short_last_chunk(N, K, B):
    """23 chunks of 48 rows and a last chunk of 1, 2 or 3 rows (a run of one
    row is its own checkpoint), in state-split teams of one and two groups."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("TEAMS", N, K, B, 12)
    rhi = min(1_000_000, cfp_r_limit(0, K))
    cost, rtab, redge = rand_case([52, N, K, B], B, N, K, 12, 10_000, 1_000_000, rlo=10_000, rhi=rhi)
    say("chunked K>256, short last chunk", N, K, B)
    assert_chain_parity(cost, rtab, redge, f"short last chunk N={N} K={K} B={B}")


@pytest.mark.parametrize("K,B", [(512, 2), (300, 5)])
def test_chunked_k512_rows_never_meet(K, B):
    """No chunk meets its checkpoints: every chunk after the first is rerun in turn."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([49, K, B])
    N = 400
    assert_form("TEAMS", N, K, B, 12)
    cost = rs.integers(0, 50, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 12, K, cfp_r_limit(0, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    say("chunked K>256, no convergence", K, B)
    assert_chain_parity(cost, rtab, redge, f"K>256 never meet K={K} B={B}")


@pytest.mark.parametrize("seed", range(4))
def test_chunked_k512_some_chunks_meet(seed):
    """Zero tables on a few edges: a seeded mix of chunks that meet in the fix-up
    pass, chunks that meet only when rerun, and chunks that never meet."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([50, seed])
    K, B, N = 512, 3, 900
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    resets = rs.choice(np.arange(1, N), size=int(rs.integers(1, 8)), replace=False)
    redge[resets] = 2
    say("chunked K>256, partial convergence", seed, sorted(resets.tolist()))
    assert_chain_parity(cost, rtab, redge, f"K>256 partial seed={seed}")


def test_teams_ignore_stale_exchange_words():
    """Batches of at most 8 searches with 256 < K <= 512 run in state-split
    teams that exchange rows as step-tagged words in the workspace.  A
    workspace of zeros (words whose tags name row 0), of all-ones, or left by
    a call on other inputs must still give the oracle's answers."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import _lib as L, search
    say("teams with stale exchange words")
    rs = np.random.default_rng(64)
    B, N, K = 3, 500, 400
    runs = []
    for _ in range(2):
        cost = rs.integers(10_000, 1_000_000, size=(B, N, K)).astype(np.int32)
        rtab = rs.integers(10_000, 1_000_000, size=(12, K, K)).astype(np.int32)
        rtab[:, np.arange(K), np.arange(K)] = 0
        redge = rs.integers(0, 12, size=N).astype(np.int32)
        o_opt, o_plan, o_st = O.chain(cost, rtab, redge, nthreads=oracle_threads())
        runs.append((dev(cost), dev(rtab), redge, o_opt, o_plan, o_st))
    nbytes = L.cfp_workspace_bytes(L.Desc(runs[0][0], runs[0][1], runs[0][2]), L.CFP_V_CHAIN)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    for fill in (0, 0xFF, 0x01):
        ws.fill_(fill)
        for j in (0, 1, 0):
            c, r, e, o_opt, o_plan, o_st = runs[j]
            res = search.dp_chain(c, r, e, ws=ws)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(res.status.cpu().numpy(), o_st, err_msg=f"status, fill {fill} input {j}")
            np.testing.assert_array_equal(res.opt.cpu().numpy(), o_opt, err_msg=f"opt, fill {fill} input {j}")
            np.testing.assert_array_equal(res.plan.cpu().numpy(), o_plan, err_msg=f"plan, fill {fill} input {j}")


def test_chunked_k512_ties_and_statuses():
    """Tie-heavy values, unavailable strategies, an infeasible search and a negative cost."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT
    cost, rtab, redge = rand_case([51], 5, 300, 512, 5, 0, 3, inf_frac=0.1)
    cost[2, 250, :] = INF   # infeasible search, in a late chunk
    assert_chain_parity(cost, rtab, redge, "chunked K>256 ties")
    cost[4, 70, 3] = -7     # a negative cost is rejected by the library
    opt, st, plan = run_chain(cost, rtab, redge)
    assert st[4] == CFP_ST_BADINPUT and opt[4] == np.iinfo(np.int64).max and (plan[4] == -1).all()
    assert st[2] != 0 and (st[[0, 1, 3]] == 0).all()


@pytest.mark.parametrize("N,K,B,E", [(1, 40, 2, 13), (3, 64, 5, 13), (47, 64, 1, 13), (84, 50, 17, 20),
                                     (500, 33, 17, 30), (400, 64, 70, 24)])
def test_chunked_many_tables(N, K, B, E):
    """More tables than the register-resident kernel holds: chains of one chunk and of
    several, four and sixteen searches per workgroup, ragged batches and blocks."""
    need_gpu()
    assert_form("WAVE", N, K, B, E)
    cost, rtab, redge = rand_case([60, N, K, B, E], B, N, K, E, 0, 1_000_000, inf_frac=0.05)
    say("chunked, many tables", N, K, B, E)
    assert_chain_parity(cost, rtab, redge, f"many tables N={N} K={K} B={B} E={E}")


@pytest.mark.parametrize("N,E", [(1, 13), (30, 70), (300, 5)])
def test_chunked_resharding_range_of_any_table(N, E):
    """A bad entry in the last table, one and several chunks, more tables than one pass of
    the packing kernel takes, on a workspace full of another call's words."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit, search
    say("chunked, R range of any table", N, E)
    cost, rtab, redge = rand_case([74, N, E], 3, N, 40, E, 0, 1000)
    bad = rtab.copy()
    bad[E - 1, 39, 39] = cfp_r_limit(0, 40)
    ws = torch.full((64 << 20,), 255, dtype=torch.uint8, device="cuda")
    for tab, want in ((rtab, 0), (bad, CFP_ST_BADINPUT), (rtab, 0)):
        r = search.dp_chain(dev(cost), dev(tab), redge, ws=ws)
        torch.cuda.synchronize()
        assert (r.status.cpu().numpy() == want).all()


@pytest.mark.parametrize("seed", range(3))
def test_chunked_some_chunks_meet_small_batch(seed):
    """Seeded patterns of chunks that do and do not meet with four searches per workgroup:
    the final pass reruns the chunks behind those that do not, up to where they meet."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([61, seed])
    K, B, N = 64, 6, 900
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    redge[rs.choice(np.arange(1, N), size=int(rs.integers(2, 12)), replace=False)] = 2
    say("chunked, partial convergence, small batch", seed)
    assert_chain_parity(cost, rtab, redge, f"partial small seed={seed}")


# K <= 32 runs with every table in LDS, chunk-parallel on long chains; a task (a chunk of
# one search) takes 16 or 32 lanes of a wave.

@pytest.mark.parametrize("N,K,B,E", [(1, 1, 1, 1), (2, 16, 5, 1), (3, 17, 3, 2), (5, 32, 9, 3), (47, 16, 4, 12),
                                     (48, 16, 4, 12), (49, 15, 7, 5), (63, 32, 2, 12), (64, 32, 2, 12),
                                     (65, 31, 1, 12), (97, 17, 33, 38), (97, 20, 3, 39), (1001, 2, 3, 4),
                                     (1000, 32, 3, 24), (203, 16, 3, 152), (64, 9, 4100, 2)])
@pytest.mark.parametrize("edges", ["random", "periodic"])
def test_narrow_shapes(N, K, B, E, edges):
    """Remainders of quads and chunks, ragged waves, tables up to and past the LDS limit
    (38 at K > 16), four and sixteen waves per workgroup, edge maps in memory and in the
    arguments."""
    need_gpu()
    assert_form("ROWS" if (K, E) == (20, 39) else "NARROW", N, K, B, E)
    cost, rtab, redge = rand_case([62, N, K, B, E], B, N, K, E, 0, 1_000_000, inf_frac=0.05)
    if edges == "periodic":
        redge = (np.arange(N) % E).astype(np.int32)
    say("narrow shape", N, K, B, E, edges)
    assert_chain_parity(cost, rtab, redge, f"narrow N={N} K={K} B={B} E={E} {edges}")


@pytest.mark.parametrize("period", [1, 5, 24, 33, 64, 65])
def test_narrow_edge_periods(period):
    """Edge maps that repeat with a period up to and past the longest one carried in the
    arguments; entry 0 (unused) breaks the pattern."""
    need_gpu()
    rs = np.random.default_rng([63, period])
    N, K, E, B = 331, 12, 9, 3
    cost, rtab, _ = rand_case([64, period], B, N, K, E, 0, 10_000)
    redge = np.resize(rs.integers(0, E, size=period), N).astype(np.int32)
    redge[0] = (redge[0] + 1) % E
    say("narrow edge period", period)
    assert_chain_parity(cost, rtab, redge, f"period {period}")


@pytest.mark.parametrize("K,B", [(32, 3), (27, 40), (16, 5), (3, 70), (18, 900), (30, 1200)])
def test_narrow_rows_never_meet(K, B):
    """Every chunk misses its checkpoints: the final pass reruns the chains; largest R."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([65, K, B])
    N = 600
    cost = rs.integers(0, 50, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 12, K, cfp_r_limit(0, K))
    redge = (np.arange(N) % 12).astype(np.int32)
    say("narrow, no convergence", K, B)
    assert_chain_parity(cost, rtab, redge, f"narrow never meet K={K} B={B}")


@pytest.mark.parametrize("N,K,B", [(1152, 27, 32), (1152, 16, 32), (700, 32, 300), (640, 20, 1100), (70, 32, 5600)])
@pytest.mark.parametrize("ratio", [1, 30])
def test_narrow_costs_that_repeat(N, K, B, ratio):
    """Costs that repeat with the edge map, so that all chunks of a search run alike: batches
    with searches none of whose chunks meets (the second fix-up, then the final pass), one,
    four and sixteen searches per workgroup of the final pass, whole and half waves per task."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([68, N, K, ratio])
    cost = rs.integers(10_000, 1_000_000, size=(B, 12, K)).astype(np.int32)[:, np.arange(N) % 12]
    rtab = rs.integers(0, min(ratio * 1_000_000, cfp_r_limit(0, K)), size=(12, K, K)).astype(np.int32)
    rtab[:, np.arange(K), np.arange(K)] = 0
    redge = (np.arange(N) % 12).astype(np.int32)
    say("narrow, repeating costs", N, K, B, ratio)
    assert_chain_parity(np.ascontiguousarray(cost), rtab, redge, f"repeating N={N} K={K} B={B} x{ratio}")


@pytest.mark.parametrize("seed", range(4))
def test_narrow_some_chunks_meet(seed):
    """Zero tables on a few edges make some chunks meet and others not, in a seeded
    pattern, with more chunks than a wave has lanes."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    rs = np.random.default_rng([66, seed])
    K, B, N = (16, 32)[seed % 2], 6, 2500
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    redge[rs.choice(np.arange(1, N), size=int(rs.integers(2, 30)), replace=False)] = 2
    say("narrow, partial convergence", seed)
    assert_chain_parity(cost, rtab, redge, f"narrow partial seed={seed}")


@pytest.mark.parametrize("N,K", [(40, 16), (40, 32), (300, 9), (300, 30)])
def test_narrow_ties_and_statuses(N, K):
    """Tie-heavy values, unavailable strategies, an infeasible search, costs 0 and 2^31 - 2
    in one row, a negative cost and an R out of range, on chains of one chunk and several."""
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit
    cost, rtab, redge = rand_case([67, N, K], 70, N, K, 5, 0, 3, inf_frac=0.1)
    cost[:, :, 0] = np.where(cost[:, :, 0] == INF, 1, cost[:, :, 0])
    cost[5, N - 7, :] = INF
    cost[6, N // 2, 1:] = 2 ** 31 - 2
    say("narrow statuses", N, K)
    assert_chain_parity(cost, rtab, redge, "narrow ties")
    cost[8, N // 3, 3] = -7
    opt, st, plan = run_chain(cost, rtab, redge)
    assert st[8] == CFP_ST_BADINPUT and opt[8] == np.iinfo(np.int64).max and (plan[8] == -1).all()
    assert st[5] == 1 and (np.delete(st, [5, 8]) == 0).all()
    rtab[3, K - 1, 2] = cfp_r_limit(0, K)
    opt, st, plan = run_chain(cost, rtab, redge)
    assert (st == CFP_ST_BADINPUT).all() and (plan == -1).all()


# 64 < K <= 128 runs chunk-parallel like the wider searches, on chains of more than 32 blocks.
# The second fix-up reruns every chunk behind one that met no checkpoint, from that one's end
# row; what still started from a wrong row then is left to the final pass.

@pytest.mark.parametrize("N,K,B,E", [(33, 65, 1, 1), (36, 128, 5, 3), (63, 128, 2, 12), (97, 100, 9, 40),
                                     (100, 127, 130, 12), (1001, 81, 3, 16), (2100, 66, 2, 12)])
def test_chunked_mid_shapes(N, K, B, E):
    """Ragged batches and last chunks, K up to 128, any number of tables."""
    need_gpu()
    assert_form("CHUNKS", N, K, B, E)
    cost, rtab, redge = rand_case([70, N, K, B], B, N, K, E, 0, 1_000_000, inf_frac=0.05)
    if N % 2:
        redge = (np.arange(N) % E).astype(np.int32)
    say("chunked mid shape", N, K, B, E)
    assert_chain_parity(cost, rtab, redge, f"chunked mid N={N} K={K} B={B} E={E}")


@pytest.mark.parametrize("K,B,N", [(100, 5, 400), (100, 90, 400), (256, 3, 400), (200, 70, 400), (400, 3, 600),
                                   (300, 9, 600), (300, 132, 200)])
@pytest.mark.parametrize("share", [0.0, 0.5, 0.8])
def test_chunked_patterns_of_unmet_chunks(K, B, N, share):
    """Zero tables near the start of a share of the chunks: isolated chunks that meet no
    checkpoint, runs of them, and (share 0) none that meets, on every chunk-parallel form
    for K > 64."""
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit
    assert_form("TEAMS" if (K, B) == (400, 3) else "CHUNKS", N, K, B, 3)
    rs = np.random.default_rng([71, K, B, int(10 * share)])
    cost = rs.integers(0, 1000, size=(B, N, K)).astype(np.int32)
    rtab = _no_switch_tables(rs, 3, K, cfp_r_limit(0, K))
    rtab[2] = 0
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    for r in range(0, N, 32 if K <= 256 else 64):
        if r and rs.random() < share:
            redge[min(N - 1, r + int(rs.integers(1, 20)))] = 2
    say("unmet patterns", K, B, share)
    assert_chain_parity(cost, rtab, redge, f"unmet K={K} B={B} share={share}")


# Where a chunk-parallel call takes longer than one that goes row after row, the latter runs:
# K > 256 below 144 rows (up to 8 searches), 352 (up to 32) or 128; 16 to 32 rows of K <= 256 run
# as two halves in batches larger than the chip. Both sides of each line, halves of odd lengths,
# and 16 tables, whose chunks grow to an even number of periods.
@pytest.mark.parametrize("N,K,B,E", [(143, 300, 8, 3), (144, 300, 8, 3), (351, 257, 9, 3), (352, 257, 9, 3),
                                     (127, 260, 33, 2), (128, 260, 33, 2), (60, 400, 12, 12), (127, 512, 4, 12),
                                     (15, 200, 300, 2), (16, 200, 300, 2), (17, 256, 257, 3), (31, 130, 270, 2),
                                     (32, 129, 300, 2), (33, 129, 300, 2), (300, 290, 5, 16)])
def test_lines_between_forms(N, K, B, E):
    need_gpu()
    cost, rtab, redge = rand_case([73, N, K, B], B, N, K, E, 0, 1_000_000, inf_frac=0.05)
    if E == 16:
        redge = (np.arange(N) % E).astype(np.int32)
    say("lines between forms", N, K, B, E)
    assert_chain_parity(cost, rtab, redge, f"lines N={N} K={K} B={B}")


@pytest.mark.parametrize("K", [100, 200, 300])
def test_chunked_repeating_costs_and_range(K):
    """Costs that repeat with the edge map, then an R out of range on a map that travels in
    the arguments and on an uploaded one, on the same workspace as a clean call."""
    need_gpu()
    import torch
    from paper_2504_00598_amd import CFP_ST_BADINPUT, cfp_r_limit, search
    rs = np.random.default_rng([72, K])
    N, B, E = 300, 3, 6
    cost = np.ascontiguousarray(rs.integers(0, 10_000, size=(B, E, K)).astype(np.int32)[:, np.arange(N) % E])
    rtab = rs.integers(0, 10_000, size=(E, K, K)).astype(np.int32)
    periodic, other = (np.arange(N) % E).astype(np.int32), rs.integers(0, E, size=N).astype(np.int32)
    bad = rtab.copy()
    bad[E - 1, K - 1, 1] = cfp_r_limit(0, K)
    say("repeating costs", K)
    o_opt, o_plan, o_st = O.chain(cost, rtab, periodic, nthreads=oracle_threads())
    r = search.dp_chain(dev(cost), dev(rtab), periodic)
    torch.cuda.synchronize()
    for _ in range(2):
        np.testing.assert_array_equal(r.status.cpu().numpy(), o_st)
        np.testing.assert_array_equal(r.opt.cpu().numpy(), o_opt)
        np.testing.assert_array_equal(r.plan.cpu().numpy(), o_plan)
        for redge in (periodic, other):
            q = search.dp_chain(dev(cost), dev(bad), redge, ws=r.ws)
            torch.cuda.synchronize()
            assert (q.status.cpu().numpy() == CFP_ST_BADINPUT).all()
        r = search.dp_chain(dev(cost), dev(rtab), periodic, ws=r.ws)
        torch.cuda.synchronize()
