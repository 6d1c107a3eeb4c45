"""GPU: the H.x of general spin by runs (narrow rows of large sectors) against
the row-by-row kernel, which takes the same vector inside a block of four FP64
columns."""
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def complete(n, count):
    """`count` bonds of the complete graph on n sites, longest first."""
    pairs = [(i, i + d, 0.25 + 0.125 * ((3 * i + d) % 7)) for d in range(n - 1, 0, -1) for i in range(n - d)]
    return pairs[:count]


def check(n, two_s, a, bonds, cols, dtype, mode=ftlm.CR, share=None):
    g, sec = ftlm.Graph(n, bonds), ftlm.Sector(n, a, mode, two_s=two_s)
    row0, nrows = share or (0, sec.dim)
    gen = torch.Generator(device="cuda").manual_seed(two_s + a)
    x = torch.randn((sec.dim, cols), dtype=dtype, device="cuda", generator=gen)
    y = torch.full((nrows, cols), 7.0, dtype=dtype, device="cuda")
    ftlm.hv_rows(sec, g, x, y, row0, nrows)
    # columns 0, 1: x; 2, 3: its magnitudes, whose product and twice the largest
    # diagonal bound the magnitudes of a row's terms
    wide = torch.empty((sec.dim, 4), dtype=torch.float64, device="cuda")
    wide[:, :2] = x.double()
    wide[:, 2:] = x.double().abs()
    want = torch.empty((nrows, 4), dtype=torch.float64, device="cuda")
    ftlm.hv_rows(sec, g, wide, want, row0, nrows)
    diag = 2 * sum(abs(J) for _, _, J in bonds) * (0.5 * two_s) ** 2
    mag = want[:, 2:] + diag * wide[row0:row0 + nrows, 2:]
    # three roundings a term (weight, product, sum) for two terms and the
    # diagonal of every bond, and those of the FP64 reference itself
    unit = 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53
    tol = 3 * (3 * len(bonds) + 2) * (unit + 2.0 ** -53) * mag[:, :cols]
    diff = (y.double() - want[:, :cols]).abs()
    assert bool((diff <= tol).all()), float((diff / tol).max())
    torch.cuda.empty_cache()


@pytest.mark.parametrize("cols,dtype", [(1, torch.float32), (2, torch.float32), (1, torch.float64)])
@pytest.mark.parametrize("n,two_s,a,mode", [(12, 4, 24, ftlm.CR), (12, 4, 22, ftlm.CLT), (14, 3, 21, ftlm.CR),
                                            (16, 2, 16, ftlm.CR), (11, 5, 27, ftlm.CR)])
def test_by_runs(n, two_s, a, mode, cols, dtype):
    bonds = graphs.icosahedron() if n == 12 else graphs.j1j2_ring(n)
    check(n, two_s, a, bonds, cols, dtype, mode)


# bonds a set of 31 holds, one more, two sets and more
@pytest.mark.parametrize("bonds", [1, 30, 31, 32, 62, 63, 66])
def test_bond_sets(bonds):
    check(12, 4, 24, complete(12, bonds), 1, torch.float32)


@pytest.mark.parametrize("share", [(0, 8388608 + 1), (5_000_001, 9_000_007), (19_611_175 - 8_400_001, 8_400_001)])
def test_shares(share):
    check(12, 4, 24, graphs.icosahedron(), 1, torch.float32, share=share)


def test_non_finite_neighbours_stay_local():
    """An infinite entry reaches its own row and its partners' rows only."""
    sec, g = ftlm.Sector(12, 24, ftlm.CR, two_s=4), ftlm.Graph(12, graphs.ring(12))
    x = torch.randn(sec.dim, device="cuda")
    x[0] = float("inf")
    y = torch.empty_like(x)
    ftlm.hv(sec, g, x, y)
    assert int((~torch.isfinite(y)).sum()) <= 1 + 2 * 12
