"""Streamed columns up to the last of 2^31 - 1 edges: positions past the end of
the range must not turn negative."""
import numpy as np
import pytest

from test_parity_gpu import mc  # noqa: F401

pytestmark = pytest.mark.gpu

M = (1 << 31) - 1


@pytest.fixture(scope="module")
def columns():
    """Successor 0 everywhere, but 4 (an accepting vertex's index) at the last edge of all."""
    import torch
    if torch.cuda.mem_get_info()[0] < 4 * M + (1 << 32):
        pytest.skip("not enough device memory")
    col = torch.zeros(M, dtype=torch.int32, device="cuda")
    col[-1] = 4
    yield col
    del col
    torch.cuda.empty_cache()


def rows(n, last):
    """Row starts of n rows of nearly equal degree, the last one of `last` edges."""
    import torch
    d = np.full(n, (M - last) // (n - 1), np.int64)
    d[:(M - last) % (n - 1)] += 1
    d[-1] = last
    start = np.concatenate([[0], np.cumsum(d)])
    assert start[-1] == M
    return torch.from_numpy(start.astype(np.int32)).cuda()


@pytest.mark.parametrize("last", [1, 300, 100_000])
def test_last_edges_of_a_small_graph(mc, columns, last):  # noqa: F811
    import torch
    n = 2048
    acc = torch.zeros(n, dtype=torch.uint8, device="cuda")
    acc[4] = 1
    csr = mc.Csr(n, M, rows(n, last), columns, None, None, None)
    batch = mc.Batch([csr], [acc])
    batch.launch()
    r = batch.read()[0]   # the last row reaches id 5, nothing reaches the last row: id 5 loses its flag
    assert r.status == 0 and r.verdict == (0, 0, 1) and r.accepting_left == 0, r


@pytest.mark.parametrize("options", ["stream", "filter"])
@pytest.mark.parametrize("last", [300, 100_000])
def test_last_edges_of_a_streamed_graph(mc, columns, last, options):  # noqa: F811
    import torch
    n = 2048
    acc = torch.zeros(n, dtype=torch.uint8, device="cuda")
    acc[4] = 1
    csr = mc.Csr(n, M, rows(n, last), columns, None, None, None)
    batch = mc.Batch([csr], [acc], gang=[256],
                     options=[mc.MAP_GRAPH_STREAM | (mc.MAP_GRAPH_FILTER if options == "filter" else 0)])
    batch.launch()
    r = batch.read()[0]
    assert r.status == 0 and r.verdict == (0, 0, 1) and r.accepting_left == 0, r
