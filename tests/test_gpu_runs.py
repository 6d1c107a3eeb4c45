"""GPU: H.x at the sizes where its kernels change (by runs or row by row, one
tile a block or a persistent grid), against the product in FP64 by an
independent index map in torch."""
import numpy as np
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


class Reference:
    """Spin-1/2 rows in FP64: a label is split in two halves, its index is the
    number of sector labels with a smaller upper half plus the rank of the lower
    half among its popcount."""

    def __init__(self, n, n_up, bonds):
        self.lo = n // 2
        nlo, nhi = 1 << self.lo, 1 << (n - self.lo)
        pc_lo, pc_hi = self.popcount(nlo), self.popcount(nhi)
        count = torch.bincount(pc_lo, minlength=n + 1)
        order = torch.argsort(pc_lo, stable=True)
        first = torch.cumsum(count, 0) - count
        self.rank = torch.empty(nlo, dtype=torch.int64, device="cuda")
        self.rank[order] = torch.arange(nlo, device="cuda") - first[pc_lo[order]]
        need = n_up - pc_hi
        rows = torch.where(need >= 0, count[need.clamp(min=0)], 0)
        self.base = torch.cumsum(rows, 0) - rows
        self.order, self.first, self.need = order, first, need
        self.bonds, self.dim = bonds, int(rows.sum())

    @staticmethod
    def popcount(count):
        x = torch.arange(count, device="cuda")
        s = torch.zeros_like(x)
        for b in range(count.bit_length()):
            s += (x >> b) & 1
        return s

    def labels(self, t):
        h = torch.searchsorted(self.base, t, right=True) - 1
        return (h << self.lo) + self.order[self.first[self.need[h]] + t - self.base[h]]

    def rows(self, x, t):
        """H x and the sum of its terms' magnitudes at the rows t."""
        lab = self.labels(t)
        x = x.double().reshape(self.dim, -1) if x.dtype != torch.float64 else x.reshape(self.dim, -1)
        out, mag = torch.zeros_like(x[t]), torch.zeros_like(x[t])
        own = x[t]
        for i, j, J in self.bonds:
            anti = ((lab >> i) ^ (lab >> j)) & 1
            m = torch.where(anti == 1, lab ^ ((1 << i) | (1 << j)), lab)
            idx = self.base[m >> self.lo] + self.rank[m & ((1 << self.lo) - 1)]
            w = (0.5 * J * anti.double())[:, None]
            d = (0.25 * J * (1.0 - 2.0 * anti.double()))[:, None]
            out += w * x[idx] + d * own
            mag += w.abs() * x[idx].abs() + d.abs() * own.abs()
        return out, mag


def dense(n, bonds):
    """A graph of n sites with `bonds` bonds of different couplings (two and three sets of bonds a lane)."""
    rng = np.random.default_rng(bonds)
    pairs = [(i, j) for i in range(n) for j in range(i + 1, n)]
    pick = rng.permutation(len(pairs))[:bonds]
    return [(pairs[k][0], pairs[k][1], float(rng.uniform(-1.0, 1.5))) for k in pick]


def check(n, n_up, bonds, cols, dtype, mode=ftlm.CR, share=None):
    g = ftlm.Graph(n, bonds)
    sec = ftlm.Sector(n, n_up, mode)
    gen = torch.Generator(device="cuda").manual_seed(n * 100 + n_up)
    x = torch.randn((sec.dim,) if cols == 1 else (sec.dim, cols), dtype=dtype, device="cuda", generator=gen)
    if share is None:
        row0, rows = 0, sec.dim
        y = torch.full_like(x, float("nan"))
        ftlm.hv(sec, g, x, y)
    else:
        row0, rows = share
        y = torch.full((rows,) + tuple(x.shape[1:]), float("nan"), dtype=dtype, device="cuda")
        ftlm.hv_rows(sec, g, x, y, row0, rows)
    assert bool(torch.isfinite(y).all()), "a row was not written"
    ref = Reference(n, n_up, bonds)
    assert ref.dim == sec.dim
    # 200,000 rows spread over the share, and its first and last rows
    t = torch.randint(rows, (200_000,), device="cuda", generator=gen)
    t = torch.cat([t, torch.arange(min(rows, 3000), device="cuda"), rows - 1 - torch.arange(min(rows, 3000), device="cuda")])
    want, mag = ref.rows(x, t + row0)
    got = y.reshape(rows, -1)[t].double()
    # at most 2 n_bonds + 3 rounded operations a row, each of the magnitude of its terms
    eps = 2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53
    assert bool(((got - want).abs() <= (2 * len(bonds) + 8) * eps * mag).all())


CLUSTER = {n: graphs.random_cluster(n, np.random.default_rng(n)) for n in (14, 16, 22, 23, 24, 25, 28)}


@pytest.mark.parametrize("n,n_up,cols,dtype", [
    (14, 7, 1, torch.float32), (16, 8, 8, torch.float32),          # few tiles: single-tile super-tiles
    (22, 11, 1, torch.float32), (23, 12, 1, torch.float32),        # on both sides of the run kernel's least rows
    (23, 12, 2, torch.float32), (24, 12, 2, torch.float32), (24, 12, 1, torch.float64),
    (24, 12, 4, torch.float32), (25, 13, 4, torch.float32), (25, 13, 2, torch.float64),
    (28, 18, 1, torch.float32), (28, 18, 2, torch.float32),        # short runs lie together
    (22, 11, 20, torch.float32), (23, 12, 12, torch.float32),      # one tile a block, with and without the LDS floor
])
def test_by_size(n, n_up, cols, dtype):
    check(n, n_up, CLUSTER[n], cols, dtype)


@pytest.mark.parametrize("bonds", [1, 62, 63, 64, 126, 127, 128])
def test_bond_sets(bonds):
    check(24, 12, dense(24, bonds), 1, torch.float32)
    check(24, 11, dense(24, bonds), 2, torch.float32)


@pytest.mark.parametrize("share", [(0, 1), (1, 255), (1_000_003, 300_007), (2_704_155, 1), (2_704_156 - 70_001, 70_001)])
def test_shares(share):
    check(24, 12, CLUSTER[24], 1, torch.float32, share=share)
    check(24, 12, CLUSTER[24], 2, torch.float32, share=share)


@pytest.mark.parametrize("mode", [ftlm.CLT, ftlm.LIN, ftlm.FULL])
@pytest.mark.parametrize("n,n_up,cols", [(16, 8, 1), (22, 11, 1), (22, 11, 4), (24, 12, 8), (25, 13, 1)])
def test_stored_maps(mode, n, n_up, cols):
    check(n, n_up, CLUSTER[n], cols, torch.float32, mode=mode)


@pytest.mark.parametrize("cols,dtype", [(1, torch.float32), (2, torch.float32)])
def test_64_bit_labels(cols, dtype):
    check(34, 10, graphs.j1j2_ring(34), cols, dtype)


@pytest.mark.parametrize("cols,dtype", [(8, torch.float32), (4, torch.float32), (2, torch.float64)])
def test_largest(cols, dtype):
    check(30, 15, graphs.icosidodecahedron(), cols, dtype)


def test_non_finite_neighbours_stay_local():
    """An infinite entry reaches its own row and its partners' rows only."""
    n, n_up = 24, 12
    bonds = CLUSTER[24]
    sec, g = ftlm.Sector(n, n_up, ftlm.CR), ftlm.Graph(n, bonds)
    x = torch.randn(sec.dim, device="cuda")
    x[0] = float("inf")
    y = torch.empty_like(x)
    ftlm.hv(sec, g, x, y)
    out = torch.empty(g.n_bonds, dtype=torch.int64, device="cuda")
    ftlm.neighbors(sec, g, 0, 1, out)
    near = set(out[out >= 0].tolist()) | {0}
    assert set(torch.nonzero(~torch.isfinite(y))[:, 0].tolist()) == near
