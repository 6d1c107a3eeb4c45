"""GPU: all chains of a tiny sector run side by side in one launch, whatever
blocks their vectors are kept in, and the tuners price that launch."""
import time

import numpy as np
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


# 20 and 64 chains are kept in several blocks, 33 in three of unlike widths
@pytest.mark.parametrize("dtype", [ftlm.F32, ftlm.F64])
@pytest.mark.parametrize("R", [11, 20, 33, 64])
def test_chains_do_not_depend_on_the_batch(R, dtype):
    g, sec = ftlm.Graph(12, graphs.j1j2_ring(12)), ftlm.Sector(12, 5, ftlm.CR)
    a, b, k = ftlm.lanczos(sec, g, 9, 0, R, 25, ftlm.GAUSS, dtype)
    for r in range(R):
        one = ftlm.lanczos(sec, g, 9, r, 1, 25, ftlm.GAUSS, dtype)
        assert np.array_equal(one[0][0], a[r]) and np.array_equal(one[1][0], b[r]) and one[2][0] == k[r]


@pytest.mark.parametrize("dtype", [ftlm.F32, ftlm.F64])
def test_plan_after_tuning(dtype):
    g = ftlm.Graph(12, graphs.j1j2_ring(12))
    plan = ftlm.Plan(g, list(range(6, 13)), ftlm.CR, 20, 20, dtype)
    want = plan.run(4, ftlm.GAUSS, use_graph=False)
    plan.tune()
    x = torch.ones(1 << 20, device="cuda")
    for use_graph in (False, True, True):
        got = plan.run(4, ftlm.GAUSS, use_graph=use_graph)
        x.mul_(1.0)
        torch.cuda.synchronize()
        assert all(np.array_equal(p, q) for p, q in zip(got, want))


# one call for all chains: a launch holds them at little more than the cost of one
@pytest.mark.parametrize("R,dtype", [(20, ftlm.F64), (24, ftlm.F32), (48, ftlm.F64)])
def test_autotune_takes_one_launch(R, dtype):
    g, sec = ftlm.Graph(12, graphs.ring(12)), ftlm.Sector(12, 6, ftlm.CR)
    t = ftlm.autotune(sec, g, R, dtype)
    assert t["batch"] == R
    assert t["candidates"][R] <= 1.5 * t["candidates"][1]


def run_us(R):
    g, sec = ftlm.Graph(12, graphs.ring(12)), ftlm.Sector(12, 6, ftlm.CR)
    work = torch.empty(ftlm.lanczos_workspace_bytes(sec, R, ftlm.F64), dtype=torch.uint8, device="cuda")
    best = 1e9
    for _ in range(20):
        torch.cuda.synchronize()
        t = time.perf_counter()
        ftlm.lanczos(sec, g, 3, 0, R, 200, ftlm.GAUSS, ftlm.F64, work=work)
        best = min(best, time.perf_counter() - t)
    return best * 1e6


def test_a_few_chains_more_take_no_second_launch():
    few, more = run_us(16), run_us(18)
    assert more <= 1.4 * few, (few, more)
