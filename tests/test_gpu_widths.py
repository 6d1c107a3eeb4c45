"""GPU: a column of a product has the same bits at every number of columns,
whichever kernels take them."""
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def check(sec, g, dtype, wide, widths):
    gen = torch.Generator(device="cuda").manual_seed(sec.dim)
    x = torch.randn((sec.dim, wide), dtype=dtype, device="cuda", generator=gen)
    want = torch.empty_like(x)
    ftlm.hv(sec, g, x, want)
    for cols in widths:
        part = x[:, -cols:].contiguous()
        y = torch.empty_like(part)
        ftlm.hv(sec, g, part, y)
        assert torch.equal(y, want[:, -cols:]), cols


# 73,789 rows at s = 1, 14,277,186 and 19,611,175 at s = 2, 144,840,476 at s = 5/2: one and two FP32
# columns and one FP64 column by runs, more of them row by row
@pytest.mark.parametrize("two_s,a", [(2, 12), (4, 20), (4, 24), (5, 30)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_general_spin(two_s, a, mode, dtype):
    g, sec = ftlm.Graph(12, graphs.icosahedron()), ftlm.Sector(12, a, mode, two_s=two_s)
    check(sec, g, dtype, 4, (1, 2, 3))
    torch.cuda.empty_cache()


# 705,432 rows (row by row), 5,200,300 and 20,058,300 (one and two columns by runs,
# more of them row by row)
@pytest.mark.parametrize("n,n_up", [(22, 11), (25, 12), (27, 13)])
@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_spin_half(n, n_up, mode, dtype):
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, n_up, mode)
    check(sec, g, dtype, 16, (1, 2, 3, 4, 5, 8, 10, 12))
    torch.cuda.empty_cache()
