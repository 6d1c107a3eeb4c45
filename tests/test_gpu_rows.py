"""GPU: FP32 Lanczos chains at the sizes where the product's work items, its
paths (row by row or by runs) and its launch widths change: a chain's
coefficients are the same bits in a block of any width as alone."""
import numpy as np
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def check(n, n_up, R, mode=ftlm.CR, bonds=None, M=3):
    bonds = bonds or graphs.random_cluster(n, np.random.default_rng(n))
    g, sec = ftlm.Graph(n, bonds), ftlm.Sector(n, n_up, mode)
    alpha, beta, steps = ftlm.lanczos(sec, g, 11, 0, R, M, ftlm.PM1, ftlm.F32)
    assert (steps == M).all() and np.isfinite(alpha).all() and np.isfinite(beta).all()
    for c in (0, R // 2, R - 1):
        a, b, _ = ftlm.lanczos(sec, g, 11, c, 1, M, ftlm.PM1, ftlm.F32)
        assert np.array_equal(alpha[c], a[0]) and np.array_equal(beta[c], b[0]), c
    torch.cuda.empty_cache()


# rows: 167960 and 125970 about 2^17 (slots of 512 and 256 rows), 705432 (two
# slots an item at the narrow widths), 1.14 and 1.35 million (one column by runs
# from 1.31), 2.7 and 5.2 million (two and four columns by runs from 2.1 and
# 4.2), 13.0 and 17.4 million about 2^24 (slots of 512 and 1024 rows), 18.2
# million with 64-bit labels, 58905 with more than 34 sites
@pytest.mark.parametrize("n,n_up", [(20, 8), (20, 9), (22, 11), (23, 10), (23, 11), (24, 12), (25, 12), (27, 11), (27, 12),
                                    (34, 8), (36, 4), (11, 5), (12, 1)])
@pytest.mark.parametrize("R", [2, 4, 8, 12, 20, 32])
def test_widths(n, n_up, R):
    check(n, n_up, R)


@pytest.mark.parametrize("mode", [ftlm.CLT, ftlm.LIN, ftlm.FULL])
@pytest.mark.parametrize("n,n_up,R", [(16, 8, 8), (22, 11, 2), (24, 12, 8), (25, 12, 4)])
def test_stored_maps(mode, n, n_up, R):
    check(n, n_up, R, mode)


@pytest.mark.parametrize("bonds", [1, 63, 64, 128])
def test_bond_sets(bonds):
    n = 24
    pairs = [(i, j, 0.25 + 0.125 * ((3 * i + j) % 7)) for d in range(1, n) for i in range(n - d) for j in [i + d]]
    check(n, 12, 8, bonds=pairs[:bonds], M=2)


def test_eight_columns_by_runs():
    check(29, 14, 8, bonds=graphs.ring(29), M=2)
