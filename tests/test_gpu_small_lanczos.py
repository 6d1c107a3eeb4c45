"""GPU: Lanczos chains of small sectors, whose items share a launch out over
waves and columns: the same bits as the same chain in a launch of any other
width."""
import numpy as np
import pytest

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def chains(sec, g, c, R, dtype, M=4):
    return ftlm.lanczos(sec, g, 7, c, R, M, ftlm.GAUSS, dtype)


# digit sums of the 12-site icosahedron: 12 and 78 rows, 1 to 5 tiles an item, on
# both sides of 256 items
@pytest.mark.parametrize("two_s,a", [(2, 1), (2, 2), (2, 8), (2, 14), (2, 12), (3, 23), (3, 26), (5, 50), (7, 70)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
@pytest.mark.parametrize("dtype", [ftlm.F32, ftlm.F64])
def test_spin_widths(two_s, a, mode, dtype):
    if mode == ftlm.CLT and two_s > 5:
        pytest.skip("a table over 8^12 labels")
    g, sec = ftlm.Graph(12, graphs.icosahedron()), ftlm.Sector(12, a, mode, two_s=two_s)
    check(sec, g, dtype)


@pytest.mark.parametrize("n,n_up", [(8, 4), (12, 6), (14, 7), (18, 7), (18, 9), (20, 10), (21, 10), (33, 4), (36, 4)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT, ftlm.LIN, ftlm.FULL])
def test_fp64_widths(n, n_up, mode):
    if n > 30 and mode != ftlm.CR:
        pytest.skip("64-bit labels have no table")
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, n_up, mode)
    check(sec, g, ftlm.F64)


def check(sec, g, dtype):
    alone = [chains(sec, g, c, 1, dtype) for c in range(16)]
    for R in (2, 4, 8, 16):
        alpha, beta, steps = chains(sec, g, 0, R, dtype)
        for c in range(R):
            assert steps[c] == alone[c][2][0]
            assert np.array_equal(alpha[c], alone[c][0][0]) and np.array_equal(beta[c], alone[c][1][0]), (R, c)

