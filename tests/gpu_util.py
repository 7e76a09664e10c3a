"""Helpers of the GPU parity tests: move seeded inputs to the device, run the
library through its C ABI binding, and compare with the oracle."""
from __future__ import annotations

import os
import sys

import numpy as np
import pytest

from oracle import oracle as O


def need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU in this container")


def oracle_threads() -> int:
    return max(1, min(16, os.cpu_count() or 1))


def dev(a, dtype=None):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.cuda()


def say(*args):
    print(*args, flush=True)
    sys.stdout.flush()


def assert_form(form, N, K, B, E):
    """A chain search of these sizes runs the kernels the test is about (a CFP_FORM_* name)."""
    from paper_2504_00598_amd import _lib as L
    assert L.cfp_chain_form(N, K, B, E) == getattr(L, "CFP_FORM_" + form), (form, N, K, B, E)


def run_chain(cost, rtab, redge):
    import torch
    from paper_2504_00598_amd import search
    res = search.dp_chain(dev(cost), dev(rtab), redge)
    torch.cuda.synchronize()
    return res.opt.cpu().numpy(), res.status.cpu().numpy(), res.plan.cpu().numpy()


def assert_chain_parity(cost, rtab, redge, label=""):
    cost = np.asarray(cost, np.int32)
    if cost.ndim == 2:
        cost = cost[None]
    g_opt, g_st, g_plan = run_chain(cost, rtab, redge)
    o_opt, o_plan, o_st = O.chain(cost, rtab, redge, nthreads=oracle_threads())
    np.testing.assert_array_equal(g_st, o_st, err_msg=f"status {label}")
    np.testing.assert_array_equal(g_opt, o_opt, err_msg=f"opt {label}")
    np.testing.assert_array_equal(g_plan, o_plan, err_msg=f"plan {label}")
    return g_opt, g_plan


def run_mem(cost, rtab, redge, mem, n_mem, budget):
    import torch
    from paper_2504_00598_amd import search
    res = search.dp_chain_mem(dev(cost), dev(rtab), redge, dev(mem), n_mem, dev(np.asarray(budget, np.int32)))
    torch.cuda.synchronize()
    return res.opt.cpu().numpy(), res.status.cpu().numpy(), res.plan.cpu().numpy()


def assert_mem_parity(cost, rtab, redge, mem, n_mem, budget, label=""):
    cost = np.asarray(cost, np.int32)
    mem = np.asarray(mem, np.uint8)
    budget = np.asarray(budget, np.int32)
    g_opt, g_st, g_plan = run_mem(cost, rtab, redge, mem, n_mem, budget)
    o_opt, o_plan, o_st = O.chain_mem(cost, rtab, redge, mem, budget, nthreads=oracle_threads())
    np.testing.assert_array_equal(g_st, o_st, err_msg=f"status {label}")
    np.testing.assert_array_equal(g_opt, o_opt, err_msg=f"opt {label}")
    np.testing.assert_array_equal(g_plan, o_plan, err_msg=f"plan {label}")
    return g_opt, g_plan


def run_frontier(cost, rtab, redge, mem, n_mem):
    import torch
    from paper_2504_00598_amd import search
    frontier, status, plan, _ = search.mem_frontier(dev(cost), dev(rtab), redge, dev(mem), n_mem)
    torch.cuda.synchronize()
    return frontier.cpu().numpy(), status.cpu().numpy(), plan.cpu().numpy()


def assert_frontier_parity(cost, rtab, redge, mem, n_mem, label=""):
    """Frontier, status and the plans at the top budget against the oracle."""
    cost = np.asarray(cost, np.int32)
    mem = np.asarray(mem, np.uint8)
    g_f, g_st, g_plan = run_frontier(cost, rtab, redge, mem, n_mem)
    o_f = O.mem_frontier(cost, rtab, redge, mem, n_mem, nthreads=oracle_threads())
    top = np.full(cost.shape[0], n_mem - 1, np.int32)
    o_opt, o_plan, o_st = O.chain_mem(cost, rtab, redge, mem, top, nthreads=oracle_threads())
    np.testing.assert_array_equal(g_st, o_st, err_msg=f"status {label}")
    np.testing.assert_array_equal(g_f, o_f, err_msg=f"frontier {label}")
    np.testing.assert_array_equal(g_f[:, -1], o_opt, err_msg=f"top budget {label}")
    np.testing.assert_array_equal(g_plan, o_plan, err_msg=f"plan {label}")
    return g_f


def run_scan(cost, rtab, redge):
    import torch
    from paper_2504_00598_amd import search
    res = search.minplus_scan(dev(cost), dev(rtab), redge)
    torch.cuda.synchronize()
    return res.opt.cpu().numpy(), res.status.cpu().numpy(), res.plan.cpu().numpy()


def assert_scan_parity(cost, rtab, redge, label=""):
    cost = np.asarray(cost, np.int32)
    if cost.ndim == 2:
        cost = cost[None]
    g_opt, g_st, g_plan = run_scan(cost, rtab, redge)
    o_opt, o_plan, o_st = O.chain(cost, rtab, redge, nthreads=oracle_threads())
    np.testing.assert_array_equal(g_st, o_st, err_msg=f"status {label}")
    np.testing.assert_array_equal(g_opt, o_opt, err_msg=f"opt {label}")
    np.testing.assert_array_equal(g_plan, o_plan, err_msg=f"plan {label}")
    return g_opt, g_plan
