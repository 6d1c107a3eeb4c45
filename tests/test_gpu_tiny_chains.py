"""GPU: chains of sectors of up to seven row tiles, whose whole run is one
launch, against the step-by-step launches that a run takes while its H.x is
timed: the same bits."""
import numpy as np
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def both(run):
    alone = run()
    ftlm.stats_enable(True)
    try:
        stepped = run()
        launches, _ = ftlm.stats_read()
    finally:
        ftlm.stats_enable(False)
        ftlm.stats_reset()
    assert launches > 0
    for p, q in zip(alone, stepped):
        assert np.array_equal(np.asarray(p), np.asarray(q))
    return alone


# 1, 12, 70, 252, 462, 924, 1287, 1716 and 1770 rows; chains that end early
@pytest.mark.parametrize("n,n_up", [(6, 6), (12, 1), (8, 4), (10, 5), (11, 5), (12, 6), (13, 5), (13, 6), (13, 7), (60, 2)])
@pytest.mark.parametrize("dtype", [ftlm.F32, ftlm.F64])
@pytest.mark.parametrize("R,M,dist", [(1, 1, ftlm.PM1), (7, 40, ftlm.GAUSS), (16, 100, ftlm.PM1)])
def test_chains(n, n_up, dtype, R, M, dist):
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, n_up, ftlm.CR)
    both(lambda: ftlm.lanczos(sec, g, 9, 3, R, min(M, sec.dim), dist, dtype))


@pytest.mark.parametrize("mode", [ftlm.CLT, ftlm.LIN, ftlm.FULL])
def test_stored_maps(mode):
    g, sec = ftlm.Graph(12, graphs.j1j2_ring(12)), ftlm.Sector(12, 6, mode)
    both(lambda: ftlm.lanczos(sec, g, 9, 0, 5, 30, ftlm.GAUSS, ftlm.F64))


@pytest.mark.parametrize("use_graph", [False, True])
def test_plan(use_graph):
    g = ftlm.Graph(12, graphs.j1j2_ring(12))
    plan = ftlm.Plan(g, list(range(6, 13)), ftlm.CR, 6, 20, ftlm.F32)
    want = both(lambda: plan.run(4, ftlm.PM1, use_graph=False))
    x = torch.ones(1 << 20, device="cuda")
    for seed in (4, 5, 4):
        got = plan.run(seed, ftlm.PM1, use_graph=use_graph)
        x.mul_(1.0)
        torch.cuda.synchronize()
        if seed == 4:
            assert all(np.array_equal(p, q) for p, q in zip(got, want))
