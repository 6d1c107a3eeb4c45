"""GPU: the row-by-row kernel on its own paths, each at sizes where no product
goes by runs: a sector's stored map, and the gathers of a single vector through
a buffer descriptor, against the gathers through pointers and the run kernel."""
import numpy as np
import pytest
import torch

from ftlm_inputs import graphs
from paper_2605_26261_amd import ftlm

pytestmark = pytest.mark.gpu


def vectors(dim, cols, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((dim, cols), dtype=dtype, device="cuda", generator=gen)


def product(sec, g, x):
    y = torch.empty_like(x)
    ftlm.hv(sec, g, x, y)
    return y


# 705,432 rows, and 14,307,150 with so few to a run that one vector is walked: rows
# of up to 8 bytes take their partners from the tables; 184,756 rows at any width
@pytest.mark.parametrize("n,n_up,cols", [(20, 10, 1), (20, 10, 8), (20, 10, 16), (22, 11, 1), (22, 11, 2), (30, 21, 1)])
def test_stored_maps_give_the_bits_of_ranking(n, n_up, cols):
    g = ftlm.Graph(n, graphs.random_cluster(n, np.random.default_rng(n)))
    x, want = None, None
    for mode in (ftlm.CR, ftlm.CLT, ftlm.LIN) + ((ftlm.FULL,) if n < 30 else ()):
        sec = ftlm.Sector(n, n_up, mode)
        x = vectors(sec.dim, cols, torch.float32, n) if x is None else x
        y = product(sec, g, x)
        want = y if want is None else want
        assert torch.equal(y, want), mode
        del sec
        torch.cuda.empty_cache()


# 16 FP64 columns take the sector's map at any size
def test_stored_maps_of_128_byte_rows():
    g = ftlm.Graph(22, graphs.j1j2_ring(22))
    x = vectors(705432, 16, torch.float64, 7)
    want = product(ftlm.Sector(22, 11, ftlm.CR), g, x)
    for mode in (ftlm.CLT, ftlm.LIN, ftlm.FULL):
        assert torch.equal(product(ftlm.Sector(22, 11, mode), g, x), want), mode


@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_buffer_gathers_equal_pointer_gathers(mode, dtype):
    """One contiguous vector goes through a buffer, a column of two through pointers."""
    n = 22
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, 11, mode)
    x = vectors(sec.dim, 2, dtype, 3)
    y = product(sec, g, x)
    one = x[:, 1].contiguous()
    assert torch.equal(product(sec, g, one), y[:, 1])
    for row0, rows in ((0, 777), (123457, 50001), (sec.dim - 333, 333)):
        part = torch.empty(rows, dtype=dtype, device="cuda")
        ftlm.hv_rows(sec, g, one, part, row0, rows)
        assert torch.equal(part, y[row0:row0 + rows, 1]), row0


@pytest.mark.parametrize("mode", [ftlm.CR, ftlm.CLT])
def test_buffer_gathers_past_two_gigabytes(mode):
    """A small share of 601,080,390 rows is walked: byte offsets up to 2.4e9 in
    32 bits. The whole product goes by runs."""
    n = 32
    g, sec = ftlm.Graph(n, graphs.j1j2_ring(n)), ftlm.Sector(n, 16, mode)
    x = vectors(sec.dim, 1, torch.float32, 5)[:, 0]
    y = torch.empty_like(x)
    ftlm.hv(sec, g, x, y)
    for row0, rows in ((0, 65_537), (sec.dim // 2, 65_537), (sec.dim - 65_537, 65_537), (sec.dim - 1, 1)):
        part = torch.empty(rows, dtype=torch.float32, device="cuda")
        ftlm.hv_rows(sec, g, x, part, row0, rows)
        assert torch.equal(part, y[row0:row0 + rows]), row0
    del sec, x, y
    torch.cuda.empty_cache()
