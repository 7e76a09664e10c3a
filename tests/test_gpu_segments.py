"""GPU parity of cfp_dp_segments + cfp_traceback_segments (segment-level
search with boundary-pair resharding) against the oracle: the chain search
over the expanded K x K tables.  Optimum, status and plan bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import dev, need_gpu, oracle_threads, say
from workloads import configs, gen

pytestmark = pytest.mark.gpu
INF = gen.COST_INF


def run_seg(cost, rbound, last, first, redge):
    import torch
    from paper_2504_00598_amd import search
    res = search.dp_segments(dev(cost), dev(rbound), dev(np.asarray(last, np.uint8)),
                             dev(np.asarray(first, np.uint8)), redge)
    torch.cuda.synchronize()
    return res.opt.cpu().numpy(), res.status.cpu().numpy(), res.plan.cpu().numpy()


def assert_seg_parity(cost, rbound, last, first, redge, label=""):
    cost = np.asarray(cost, np.int32)
    if cost.ndim == 2:
        cost = cost[None]
    g_opt, g_st, g_plan = run_seg(cost, rbound, last, first, redge)
    o_opt, o_plan, o_st = O.segments(cost, rbound, last, first, redge, nthreads=oracle_threads())
    np.testing.assert_array_equal(g_st, o_st, err_msg=f"status {label}")
    np.testing.assert_array_equal(g_opt, o_opt, err_msg=f"opt {label}")
    np.testing.assert_array_equal(g_plan, o_plan, err_msg=f"plan {label}")
    return g_opt, g_plan


def assert_form(form, N, K, B, E, L, F):
    """A call of these sizes runs the kernels the test is about: over boundary CLASSes, or
    over plans in CHUNKS or all ROWS at once."""
    from paper_2504_00598_amd import _lib
    assert _lib.cfp_segment_form(N, K, B, E, L, F) == getattr(_lib, "CFP_FORM_SEG_" + form), (form, N, K, B, E, L, F)


# Sizes of each form: searches past the class form's memory limit, batches past its line
FORMS = [("CLASS", 8, 40), ("CHUNKS", 8, 1500), ("ROWS", 800, 40)]


def seg_case(seed, B, N, P, S, E, lo, hi):
    rs = np.random.default_rng(seed)
    K = S ** P
    last, first = gen.digit_maps(P, S)
    cost = rs.integers(lo, hi, size=(B, N, K)).astype(np.int32)
    # boundary entries inside the exact range for this K (2^23 - 1 at K = 512)
    rhi = min(hi, (1 << (32 - max(4, int(np.ceil(np.log2(K)))))) - 1)
    rbound = rs.integers(min(lo, rhi - 1), rhi, size=(E, S, S)).astype(np.int32)
    redge = rs.integers(0, E, size=N).astype(np.int32)
    return cost, rbound, last, first, redge


def test_config_full():
    need_gpu()
    say("config seg_gpt_n96_k81")
    d = configs.make("seg_gpt_n96_k81")
    assert_seg_parity(d["cost"], d["rbound"], d["last"], d["first"], d["redge"], "seg config")


# K = S^P from 2 to 512 with up to 4 or up to 8 boundary strategies
@pytest.mark.parametrize("N,P,S", [(1, 1, 2), (2, 1, 5), (5, 2, 3), (50, 4, 3), (30, 3, 4), (20, 5, 2), (40, 4, 4),
                                   (10, 2, 8), (8, 3, 8), (70, 2, 7), (25, 3, 6), (12, 9, 2), (9, 4, 3),
                                   (17, 2, 3)])
def test_shapes(N, P, S):
    need_gpu()
    say("seg shape", N, P, S)
    cost, rbound, last, first, redge = seg_case([N, P, S], 5, N, P, S, 3, 10_000, 10_000_000)
    assert_seg_parity(cost, rbound, last, first, redge, f"N={N} P={P} S={S}")


def test_general_maps_unequal_boundaries():
    """Arbitrary plan-to-boundary maps with different strategy counts on the
    two sides (L = 3 last-block strategies, F = 5 first-block ones)."""
    need_gpu()
    rs = np.random.default_rng(77)
    B, N, K, L, F = 6, 60, 100, 3, 5
    last = rs.integers(0, L, size=K).astype(np.uint8)
    first = rs.integers(0, F, size=K).astype(np.uint8)
    cost = rs.integers(0, 10**6, size=(B, N, K)).astype(np.int32)
    rbound = rs.integers(0, 10**6, size=(4, L, F)).astype(np.int32)
    redge = rs.integers(0, 4, size=N).astype(np.int32)
    assert_seg_parity(cost, rbound, last, first, redge, "general maps")


@pytest.mark.parametrize("S", [2, 3])
@pytest.mark.parametrize("form,B,N", FORMS)
def test_heavy_ties(S, form, B, N):
    need_gpu()
    assert_form(form, N, S ** 4, B, 2, S, S)
    say("seg ties", S, form)
    cost, rbound, last, first, redge = seg_case([9, S], B, N, 4, S, 2, 0, 3)
    assert_seg_parity(cost, rbound, last, first, redge, f"ties S={S} {form}")


@pytest.mark.parametrize("form,B,N", FORMS)
def test_unavailable_and_statuses(form, B, N):
    need_gpu()
    from paper_2504_00598_amd import CFP_ST_BADINPUT, CFP_ST_INFEASIBLE, cfp_r_limit, CFP_V_SEG
    assert_form(form, N, 81, B, 2, 3, 3)
    say("seg statuses", form)
    cost, rbound, last, first, redge = seg_case(10, B, N, 4, 3, 2, 0, 1000)
    cost[0][cost[0] % 4 == 0] = INF
    cost[1, 7, :] = INF                     # no plan
    cost[2, 3, 5] = -1                      # negative cost
    opt, st, plan = run_seg(cost, rbound, last, first, redge)
    assert st[1] == CFP_ST_INFEASIBLE and st[2] == CFP_ST_BADINPUT
    assert (plan[1] == -1).all() and (plan[2] == -1).all()
    good = np.delete(cost, [1, 2], axis=0)
    assert_seg_parity(good, rbound, last, first, redge, f"inf {form}")
    # boundary entry at the exact-range limit, and a map entry out of range
    rb = rbound.copy()
    rb[1, 2, 0] = cfp_r_limit(CFP_V_SEG, 81)
    _, st, _ = run_seg(good, rb, last, first, redge)
    assert (st == CFP_ST_BADINPUT).all()
    bad_last = last.copy()
    bad_last[17] = 3
    _, st, _ = run_seg(good, rbound, bad_last, first, redge)
    assert (st == CFP_ST_BADINPUT).all()
    bad_first = first.copy()
    bad_first[80] = 3
    _, st, _ = run_seg(good, rbound, last, bad_first, redge)
    assert (st == CFP_ST_BADINPUT).all()


@pytest.mark.parametrize("form,B,N", FORMS)
def test_max_boundary_values(form, B, N):
    need_gpu()
    from paper_2504_00598_amd import cfp_r_limit, CFP_V_SEG
    assert_form(form, N, 81, B, 2, 3, 3)
    say("seg max boundary", form)
    cost, rbound, last, first, redge = seg_case(11, B, N, 4, 3, 2, 0, 10**7)
    rbound[:] = cfp_r_limit(CFP_V_SEG, 81) - 1
    rbound[:, np.arange(3), np.arange(3)] = 0
    assert_seg_parity(cost, rbound, last, first, redge, "max r")


def test_repeat_is_bit_identical():
    need_gpu()
    d = configs.make("seg_gpt_n96_k81", batch=32)
    a = run_seg(d["cost"], d["rbound"], d["last"], d["first"], d["redge"])
    for _ in range(3):
        b = run_seg(d["cost"], d["rbound"], d["last"], d["first"], d["redge"])
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


# Calls that do not run over classes (more than 768 searches, few classes of many plans,
# chains past the class form's memory limit) run over plans: batches that leave SIMDs idle
# as chunks (rank convergence), one workgroup per search, P = min(8, 1024 // B, N // 16)
# chunks of ceil(N / P) rows; others one wave per search.
def seg_chunks(N, B):
    P = min(8, max(1, 1024 // B), N // 16)
    return P if P >= 2 else 1


@pytest.mark.parametrize("B,N,K,L,F", [(2, 700, 64, 1, 2), (2, 470, 30, 6, 7), (2, 300, 128, 2, 2), (2, 300, 125, 5, 1),
                                       (4, 200, 216, 2, 2), (4, 450, 216, 6, 6), (2, 200, 250, 1, 6), (3, 70, 512, 2, 2),
                                       (3, 80, 512, 8, 2), (3, 450, 300, 8, 8), (2, 1500, 81, 3, 3)])
def test_chunked_shapes_across_kernel_forms(B, N, K, L, F):
    """One, two, four and eight states per lane (K up to 64, 128, 256 and 512, the last with
    16-bit argmins) with up to 4 and up to 8 boundary strategies."""
    need_gpu()
    assert_form("CHUNKS", N, K, B, 3, L, F)
    _plans_case([70, N, K], B, N, K, L, F)


@pytest.mark.parametrize("B,N,K,L,F", [(780, 1, 40, 3, 3), (780, 9, 50, 3, 3), (780, 9, 50, 8, 5), (780, 17, 100, 4, 2),
                                       (780, 12, 120, 5, 6), (800, 12, 200, 3, 3), (800, 9, 216, 6, 6),
                                       (770, 10, 512, 2, 2), (780, 9, 512, 8, 8)])
def test_one_wave_per_search(B, N, K, L, F):
    """The same without chunks; N = 9 and 17 end one row into a group of 8 steps."""
    need_gpu()
    assert_form("ROWS", N, K, B, 3, L, F)
    _plans_case([75, N, K], B, N, K, L, F)


def _plans_case(seed, B, N, K, L, F):
    say("seg over plans", B, N, K, L, F)
    rs = np.random.default_rng(seed)
    last, first = rs.integers(0, L, size=K).astype(np.uint8), rs.integers(0, F, size=K).astype(np.uint8)
    cost = rs.integers(10_000, 10_000_000, size=(B, N, K)).astype(np.int32)
    cost[rs.random((B, N, K)) < 0.1] = INF
    cost[:, :, K - 1] = np.where(cost[:, :, K - 1] == INF, 9, cost[:, :, K - 1])
    rbound = rs.integers(10_000, 8_000_000, size=(3, L, F)).astype(np.int32)
    redge = rs.integers(0, 3, size=N).astype(np.int32)
    assert_seg_parity(cost, rbound, last, first, redge, f"plans B={B} N={N} K={K} L={L} F={F}")


def _class_chains(seed, B, N, E_mix, pattern, K=12):
    """Plans whose first and last block strategies coincide (first = last = s mod 3) and
    boundary table 0 that never moves a search between classes (0 on the diagonal, the
    largest entry off it): over rows using table 0 the three classes run as separate
    chains, so a run started anywhere else never becomes parallel to the true one.  The
    other tables mix the classes.  pattern[p] says whether chunk p's rows use table 0 (the
    pattern repeats where there are more chunks)."""
    from paper_2504_00598_amd import cfp_r_limit, CFP_V_SEG
    rs = np.random.default_rng(seed)
    L = 3
    last = (np.arange(K) % L).astype(np.uint8)
    first = last.copy()
    cost = rs.integers(0, 10**6, size=(B, N, K)).astype(np.int32)
    rbound = rs.integers(0, 10**5, size=(1 + E_mix, L, L)).astype(np.int32)
    rbound[0] = cfp_r_limit(CFP_V_SEG, K) - 1
    rbound[0][np.arange(L), np.arange(L)] = 0
    P = seg_chunks(N, B)
    CL = -(-N // P)
    redge = rs.integers(1, 1 + E_mix, size=N).astype(np.int32)
    for p in range(P):
        if pattern[p % len(pattern)]:
            redge[p * CL:min((p + 1) * CL, N)] = 0
    return cost, rbound, last, first, redge, P


# the chunked form at one, two, four and eight states per lane: chains past the class
# form's limit, and more plans per class than it takes
CHUNKED = [(1600, 12), (1450, 100), (160, 230), (120, 300)]


@pytest.mark.parametrize("N,K", CHUNKED)
def test_chunked_rows_that_never_meet(N, K):
    """Every row's table keeps the classes apart: no fix-up meets its chunk's
    speculative rows, and the final pass reruns every chunk after the first."""
    need_gpu()
    assert_form("CHUNKS", N, K, 4, 3, 3, 3)
    say("seg chunks never meet", N, K)
    cost, rbound, last, first, redge, P = _class_chains(71, 4, N, 2, [True], K)
    assert P >= 4
    assert_seg_parity(cost, rbound, last, first, redge, f"never meet N={N} K={K}")


@pytest.mark.parametrize("N,K", CHUNKED)
@pytest.mark.parametrize("pattern", [(False, True, False, False), (False, True, True, False),
                                     (True, False, True, False), (False, False, False, True)])
def test_chunked_rows_that_meet_in_some_chunks(pattern, N, K):
    """A chunk of class-separating rows leaves its successor's fix-up started from a
    wrong row: that chunk is rerun from the true row, at least as far as its fix-up
    went, and where the rerun meets the speculative rows the chunks after it count
    again; two such chunks in a row chain the reruns."""
    need_gpu()
    assert_form("CHUNKS", N, K, 4, 3, 3, 3)
    say("seg chunks meet in some", pattern, N, K)
    cost, rbound, last, first, redge, P = _class_chains([72, *pattern], 4, N, 2, pattern, K)
    assert P >= 4
    assert_seg_parity(cost, rbound, last, first, redge, f"pattern {pattern} N={N} K={K}")


@pytest.mark.parametrize("B,N,P,S,form", [(3, 1600, 2, 3, "CHUNKS"), (3, 1536, 2, 3, "CHUNKS"), (520, 1600, 2, 2, "ROWS"),
                                          (800, 50, 2, 3, "ROWS"), (3, 90, 2, 3, "CLASS")])
def test_edge_map_in_arguments_and_in_workspace(B, N, P, S, form):
    """Over plans, chains of up to 1536 segments carry their edge map in the kernel
    arguments; longer ones read the device copy uploaded with the header.  Both,
    chunked (small batch) and one wave per search; over classes a map without a
    period is uploaded."""
    need_gpu()
    assert_form(form, N, S ** P, B, 5, S, S)
    say("seg edge map", B, N, P, S)
    cost, rbound, last, first, redge = seg_case([73, B, N], B, N, P, S, 5, 10_000, 10_000_000)
    assert_seg_parity(cost, rbound, last, first, redge, f"B={B} N={N} K={S ** P}")


# Searches whose class minima fit in LDS (about 1400 segments with up to four boundary
# strategies, 400 with more) run the recurrence over boundary classes, other than the
# large batches and large classes above.

@pytest.mark.parametrize("N,K,L,F,E,B", [(1, 5, 1, 1, 1, 3), (2, 3, 8, 8, 1, 2), (3, 512, 8, 1, 2, 2),
                                         (17, 512, 1, 8, 3, 3), (40, 100, 5, 2, 200, 2), (33, 7, 4, 4, 3, 5),
                                         (300, 64, 3, 4, 5, 600), (1390, 9, 3, 3, 4, 2), (1450, 9, 3, 3, 4, 2),
                                         (380, 30, 6, 7, 4, 2), (470, 30, 6, 7, 4, 2), (20, 50, 3, 3, 3000, 2)])
def test_class_form_shapes(N, K, L, F, E, B):
    """Arbitrary maps (empty classes, more classes than plans), unequal boundaries, many
    tables (3000 past what LDS holds), chains on both sides of its limit; costs over the whole range in some
    rows, plans and whole classes that are not available."""
    need_gpu()
    assert_form("CHUNKS" if N in (1450, 470) else "ROWS" if E == 3000 else "CLASS", N, K, B, E, L, F)
    from paper_2504_00598_amd import cfp_r_limit, CFP_V_SEG
    say("segment classes", N, K, L, F, E, B)
    rs = np.random.default_rng([90, N, K, L, F])
    last = rs.integers(0, L, size=K).astype(np.uint8)
    first = rs.integers(0, F, size=K).astype(np.uint8)
    cost = rs.integers(0, 100_000, size=(B, N, K)).astype(np.int32)
    wide = rs.random((B, N)) < 0.1
    cost[wide] = rs.integers(0, 2 ** 31 - 1, size=(int(wide.sum()), K))
    gone = rs.random((B, N, F)) < 0.2                       # whole first classes
    cost[gone[:, :, first]] = INF
    cost[:, :, K // 2] = np.where(cost[:, :, K // 2] == INF, 77, cost[:, :, K // 2])
    rbound = rs.integers(0, cfp_r_limit(CFP_V_SEG, K), size=(E, L, F)).astype(np.int32)
    redge = rs.integers(0, E, size=N).astype(np.int32)
    assert_seg_parity(cost, rbound, last, first, redge, f"classes N={N} K={K} L={L} F={F}")


@pytest.mark.parametrize("L,F", [(3, 3), (6, 5)])
def test_class_form_ties(L, F):
    """Values in {0, 1}: the lowest plan over every tied class and boundary."""
    need_gpu()
    rs = np.random.default_rng([91, L, F])
    B, N, K = 6, 90, 60
    cost = rs.integers(0, 2, size=(B, N, K)).astype(np.int32)
    rbound = rs.integers(0, 2, size=(3, L, F)).astype(np.int32)
    last, first = rs.integers(0, L, size=K).astype(np.uint8), rs.integers(0, F, size=K).astype(np.uint8)
    redge = np.resize(np.array([1, 2, 0, 1, 1], np.int32), N)
    redge[:3] = [2, 2, 0]  # a head of its own before the period
    say("segment class ties", L, F)
    assert_seg_parity(cost, rbound, last, first, redge, f"class ties L={L} F={F}")


@pytest.mark.parametrize("pattern", [(True,) * 8, (False, True, False, False, True, True, False, False)])
def test_long_chains_that_meet_in_some_chunks(pattern):
    """Eight chunks, on chains past the class form's limit: chunks that never meet and
    patterns of those that do."""
    need_gpu()
    assert_form("CHUNKS", 1600, 12, 4, 3, 3, 3)
    say("long segment chunks", pattern)
    cost, rbound, last, first, redge, P = _class_chains([92, *pattern], 4, 1600, 2, pattern)
    assert P == 8
    assert_seg_parity(cost, rbound, last, first, redge, f"long pattern {pattern}")


@pytest.mark.parametrize("N,K,L,F,B,most", [(40, 512, 8, 8, 3, 440), (40, 512, 1, 1, 3, 512), (1, 300, 1, 1, 2, 300),
                                            (60, 130, 2, 2, 5, 100), (33, 77, 4, 3, 4, 70), (25, 512, 5, 6, 3, 60),
                                            (200, 20, 1, 1, 3, 20), (9, 509, 8, 1, 2, 300)])
@pytest.mark.parametrize("hi", [3, 2 ** 31 - 1])
def test_class_form_uneven_maps(N, K, L, F, B, most, hi):
    """One class with most of the plans, spread over the plan indices: the lanes share the
    plans evenly; ties, unavailable strategies, the whole cost range, a negative cost."""
    need_gpu()
    assert_form("CLASS", N, K, B, 2, L, F)
    from paper_2504_00598_amd import CFP_ST_BADINPUT
    say("segment uneven maps", N, K, L, F, B, hi)
    rs = np.random.default_rng([93, N, K, L, F])
    last, first = rs.integers(0, L, size=K).astype(np.uint8), rs.integers(0, F, size=K).astype(np.uint8)
    big = rs.choice(K, size=most, replace=False)
    last[big], first[big] = L - 1, 0
    cost = rs.integers(0, hi, size=(B, N, K), dtype=np.int64).astype(np.int32)
    cost[rs.random((B, N, K)) < 0.3] = INF
    cost[:, :, K // 3] = np.where(cost[:, :, K // 3] == INF, 1, cost[:, :, K // 3])
    rbound = rs.integers(0, min(hi, 1000), size=(2, L, F)).astype(np.int32)
    redge = rs.integers(0, 2, size=N).astype(np.int32)
    assert_seg_parity(cost, rbound, last, first, redge, f"uneven N={N} K={K} L={L} F={F}")
    cost[0, N // 2, big[0]] = -3
    _, st, plan = run_seg(cost, rbound, last, first, redge)
    assert st[0] == CFP_ST_BADINPUT and (plan[0] == -1).all() and (st[1:] == 0).all()


@pytest.mark.parametrize("B,N,K,L,F,form", [
    (768, 20, 30, 3, 3, "CLASS"), (769, 20, 30, 3, 3, "ROWS"), (800, 60, 216, 6, 6, "CLASS"),
    (800, 40, 216, 6, 6, "ROWS"), (5, 512, 64, 1, 1, "CLASS"), (5, 513, 64, 1, 1, "CHUNKS"),
    (2, 140, 240, 3, 3, "CHUNKS"), (2, 136, 240, 3, 3, "CLASS")])
def test_lines_between_forms(B, N, K, L, F, form):
    """Both sides of the lines by batch and by plans per class."""
    need_gpu()
    assert_form(form, N, K, B, 3, L, F)
    say("segment lines", B, N, K, L, F)
    rs = np.random.default_rng([94, B, N, K])
    last, first = rs.integers(0, L, size=K).astype(np.uint8), rs.integers(0, F, size=K).astype(np.uint8)
    cost = rs.integers(0, 10**6, size=(B, N, K)).astype(np.int32)
    cost[rs.random((B, N, K)) < 0.1] = INF
    cost[:, :, 0] = np.where(cost[:, :, 0] == INF, 9, cost[:, :, 0])
    rbound = rs.integers(0, 10**6, size=(3, L, F)).astype(np.int32)
    redge = rs.integers(0, 3, size=N).astype(np.int32)
    assert_seg_parity(cost, rbound, last, first, redge, f"lines B={B} N={N} K={K}")
