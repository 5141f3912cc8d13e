"""A server's device memory stays within its budget across evictions: what cached
operator sets and solve state hold, and what earlier ones left idle for reuse.
Operators of two sizes, so that the blocks of one size stay behind when the
other's sets take their place."""
import time

import numpy as np
import pytest
import torch

import workloads as wl
from paper_1805_08990_amd import _binding as b
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu

MIB = 1 << 20
K = 2  # quadrature nodes, each with a dense exponential of a nonsymmetric operator


def _run(srv, op, n):
    opts = b.SolveOptions(T=0.02, h=0.01, tol=1e-10, quad_nodes=K, max_rank=32)
    t, t0 = srv.submit(op, "dle", opts, wl.random_C(1, n, n), n), time.time()
    while (r := srv.poll(t)) is None:
        assert time.time() - t0 < 60
        time.sleep(0.001)
    return np.array(r[0]), np.array(r[1])


def test_held_memory_within_budget(ctx):
    sizes = [2048] * 5 + [1856] * 6 + [2048] * 2
    ops = []
    for i, n in enumerate(sizes):
        rng = np.random.default_rng(i)
        A = rng.standard_normal((n, n)) / np.sqrt(n)
        A[np.arange(n), np.arange(n)] -= 3.0
        ops.append(ctx.register_operator(A))
    warm = ctx.server(8 << 30, max_slots=1)  # the kernels' code and the runtime's own memory
    want = [_run(warm, ops[0], sizes[0]), _run(warm, ops[5], sizes[5])]
    warm.stop()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    # four sets of the larger size and a solve's state
    budget = 4 * (K + 1) * 8 * 2048 ** 2 + 48 * MIB
    free0 = torch.cuda.mem_get_info()[0]
    srv = ctx.server(budget, max_slots=1)
    try:
        for i, n in enumerate(sizes):
            L, D = _run(srv, ops[i], n)
            got = free0 - torch.cuda.mem_get_info()[0]
            announce("server budget", i, n, f"held {got / MIB:.0f} MiB of {budget / MIB:.0f}")
            assert np.isfinite(L).all() and np.isfinite(D).all()
            # 2 MiB pages: up to 1.7 MiB a block of the smaller size; 16 MiB for the runtime
            assert got <= budget + (K + 1) * 5 * 2 * MIB + 16 * MIB
        assert srv.stats()["peak_bytes"] <= budget
        for i, w in zip((0, 5), want):  # evicted meanwhile: built again, the same
            assert all(np.array_equal(x, y) for x, y in zip(_run(srv, ops[i], sizes[i]), w))
    finally:
        srv.stop()
