"""GPU: an infinity or a NaN in x reaches the products' rows that have it as a
term and no others, whichever kernel and index map a product takes."""
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def check(sec, g, cols, dtype):
    terms = g.n_bonds * (2 if sec.two_s > 1 else 1)
    far = sec.dim // 2 + 1
    x = torch.randn((sec.dim, cols), dtype=dtype, device="cuda")
    x[0, 0] = float("inf")
    x[far, cols - 1] = float("nan")
    y = torch.empty_like(x)
    ftlm.hv(sec, g, x, y)
    want = [set() for _ in range(cols)]
    for row, col in ((0, 0), (far, cols - 1)):
        out = torch.empty(terms, dtype=torch.int64, device="cuda")
        ftlm.neighbors(sec, g, row, 1, out)
        want[col] |= set(out[out >= 0].tolist()) | {row}
    for col in range(cols):
        got = torch.nonzero(~torch.isfinite(y[:, col]))[:, 0].cpu()
        assert torch.equal(got, torch.tensor(sorted(want[col]))), (cols, col, len(got), len(want[col]))


# 48,620 rows (every map its own), 705,432 (ranked in place of a map from eight
# bytes a row on), 5,200,300 (one to four columns by runs)
@pytest.mark.parametrize("n,n_up", [(18, 9), (22, 11), (25, 12)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT, ftlm.LIN, ftlm.FULL])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_spin_half(n, n_up, mode, dtype):
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, n_up, mode)
    for cols in (1, 2, 4, 8, 16):
        check(sec, g, cols, dtype)


# 73,789 rows, and 19,611,175 (one and two columns by runs)
@pytest.mark.parametrize("two_s,a", [(2, 12), (4, 24)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_general_spin(two_s, a, mode, dtype):
    g, sec = ftlm.Graph(12, graphs.ring(12)), ftlm.Sector(12, a, mode, two_s=two_s)
    for cols in (1, 2, 4):
        check(sec, g, cols, dtype)
