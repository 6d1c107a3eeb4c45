"""GPU: Lanczos runs in sectors of many sites: their time, and the same bits at
every number of chains."""
import time

import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def run(n, n_up, R, M, dtype=ftlm.F32, best_of=1):
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, n_up, ftlm.CR)
    work = torch.empty(ftlm.lanczos_workspace_bytes(sec, R, dtype), dtype=torch.uint8, device="cuda")
    best = float("inf")
    for _ in range(best_of):
        t = time.perf_counter()
        alpha, beta, steps = ftlm.lanczos(sec, g, 7, 0, R, M, ftlm.PM1, dtype, work=work)
        best = min(best, time.perf_counter() - t)
    return alpha, beta, steps, best / sec.dim


# with room for any binomial table beside its Y values a workgroup of 62 sites would
# not fit a CU's LDS twice: a row takes 1.1 times as long as one of 61 sites, 1.9 then
def test_62_sites_take_little_longer_than_61():
    t62, t61 = (run(n, 5, 8, 10, best_of=5)[3] for n in (62, 61))
    assert t62 <= 1.4 * t61, (t62, t61)


# 20 columns in one launch take twice as long as 8, three times as 8, 8 and 4
def test_20_columns_take_little_longer_than_8():
    t20, t8 = (run(47, 41, R, 8, best_of=4)[3] for R in (20, 8))
    assert t20 <= 2.4 * t8, (t20, t8)


# 376,992, 850,668 and 22,100 rows: whichever launches take a chain, it has the same bits
@pytest.mark.parametrize("n,n_up", [(36, 31), (42, 5), (52, 3)])
@pytest.mark.parametrize("dtype", [ftlm.F32, ftlm.F64])
def test_same_bits(n, n_up, dtype):
    most = run(n, n_up, 33, 6, dtype)
    for R in (1, 8, 12, 16, 20, 23, 32):
        some = run(n, n_up, R, 6, dtype)
        for a, b in zip(some[:3], most[:3]):
            assert (a == b[:R]).all(), R


# two columns take 1.05 times as long as one, 1.4 times by runs
def test_few_columns_above_32_sites():
    two, one = (run(34, 10, R, 6, best_of=3)[3] for R in (2, 1))
    torch.cuda.empty_cache()
    assert two <= 1.25 * one, (two, one)
