"""Filtered sweeps at the edges of the rules that choose their form by size,
bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle
import synth
from test_parity_gpu import check_detect, mc  # noqa: F401

pytestmark = pytest.mark.gpu

BANDS = 3 << 21   # vertices from which one-way graphs are swept in bands


def one_way(n, up, wrong=0):
    """Vertex v >= 2 has 1..4 edges to lower ids (higher, mirrored, where up); `wrong` edges more the other way."""
    rng = np.random.default_rng(n + wrong)
    src = np.repeat(np.arange(2, n + 1, dtype=np.int64), rng.integers(1, 5, n - 1))
    dst = 1 + rng.integers(0, 1 << 62, src.size) % (src - 1)
    if wrong:
        i = rng.choice(src.size, wrong, replace=False)
        src, dst = np.concatenate([src, dst[i]]), np.concatenate([dst, np.minimum(n, dst[i] + 1 + i % 1000)])
    if up:
        src, dst = n + 1 - src, n + 1 - dst
    acc = np.zeros(n, np.uint8)
    acc[rng.choice(n, n // 700, replace=False)] = 1
    return synth.Graph(n=n, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=acc,
                       name=f"one-way(n={n},up={up},wrong={wrong})")


@pytest.mark.parametrize("n,up,wrong", [(BANDS - 1, False, 0), (BANDS, True, 0), (BANDS + 33, False, 20_000),
                                        (BANDS + 4097, False, 30), (BANDS + 70_001, True, 1_000_000)])
def test_bands_by_size(mc, n, up, wrong):  # noqa: F811
    g = one_way(n, up, wrong)
    ref = oracle.map_detect(g, mode="desc", maps_cap=1)
    csr = mc.build_csr(g.n, g.src, g.dst)
    for flags in (mc.MAP_FLAG_DIRECTION, 0):
        check_detect(mc, g, csr, flags=flags, ref=ref)
        got, res = mc.propagate(csr, g.acc, flags=flags)
        assert res.status == 0 and np.array_equal(got.cpu().numpy(), ref.maps[0])


PUSH_ROWS = (1 << 13, 1 << 16)   # rows of a workgroup from which a reset may push, and from which n / 8 rows may


def test_push_share_by_rows(mc):  # noqa: F811
    """One workgroup per graph, with rows and accepting vertices on both sides of the lines."""
    graphs, opts = [], []
    for rows in PUSH_ROWS:
        for n in (rows - 65, rows - 1, rows, rows + 1, rows + 63):
            for k in (n // 16 - 1, n // 16 + 1, n // 8 - 1, n // 8 + 1):
                g = one_way(n, (n + k) & 1 == 0, wrong=64 if k & 1 else 0)
                g.acc[:] = 0
                g.acc[np.random.default_rng(k).choice(n, k, replace=False)] = 1
                graphs.append(g)
    csrs = [mc.build_csr(g.n, g.src, g.dst) for g in graphs]
    opts = [mc.MAP_GRAPH_FILTER | mc.MAP_GRAPH_DIRECTION | mc.MAP_GRAPH_STREAM] * len(graphs)
    batch = mc.Batch(csrs, [g.acc for g in graphs], options=opts)
    for _ in range(2):
        batch.launch()
        for g, r in zip(graphs, batch.read()):
            ref = oracle.map_detect(g, mode="desc")
            assert r.status == 0 and r.verdict == ref.verdict and r.accepting_left == ref.accepting_left, (g.name, r)


@pytest.mark.parametrize("direction", [False, True], ids=["pull", "direction-switch"])
@pytest.mark.parametrize("n", [1, 5, 63, 4096, 5003, 16_383, 16_384, 16_385, 33_003, 133_001, 300_007, 524_288, 524_289])
def test_few_rows_per_wave(mc, n, direction):  # noqa: F811
    """Streamed graphs of a tile or two per wave, rows not a multiple of anything, bitmaps at the sizes where they
    are read in place, copied and folded."""
    g = one_way(n, n % 2 == 0, wrong=n // 50) if n > 1 else synth.from_edges(1, [(1, 1)], [1], "loop")
    if n > 700:
        g.acc[n // 3:n // 3 + n // 40] = 1
    csr = mc.build_csr(g.n, g.src, g.dst)
    flags = mc.MAP_FLAG_STREAM | (mc.MAP_FLAG_DIRECTION if direction else 0)
    ref = oracle.map_detect(g, mode="desc", maps_cap=1)
    check_detect(mc, g, csr, flags=flags, ref=ref)
    if len(ref.maps):
        got, res = mc.propagate(csr, g.acc, flags=flags)
        assert res.status == 0 and np.array_equal(got.cpu().numpy(), ref.maps[0])
