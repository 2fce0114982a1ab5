"""Filtered stream sweeps against the CPU oracle, bit-exact: sizes around the batches of rows that a pass takes,
accepting sets on both sides of the size below which they push their ids into freshly reset rows, runs that end
because no accepting vertex is left, capped runs, propagation."""
import numpy as np
import pytest

import synth
from test_parity_gpu import check_detect, check_propagate_all, mc  # noqa: F401

pytestmark = pytest.mark.gpu


def graph(n, k, up, seed, cycle=False):
    """Random graph with about 3 edges per vertex to higher (up) or lower ids and k accepting vertices."""
    g = synth.random_graph(seed, n, 3 * n, p_acc=0.0)
    lo, hi = np.minimum(g.src, g.dst), np.maximum(g.src, g.dst)
    keep = lo != hi
    src, dst = (lo[keep], hi[keep]) if up else (hi[keep], lo[keep])
    acc = np.zeros(n, np.uint8)
    acc[np.random.default_rng(seed).choice(n, min(n, k), replace=False)] = 1
    if cycle and src.size:
        src, dst = np.append(src, dst[-1]), np.append(dst, src[-1])
    return synth.Graph(n=n, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=acc,
                       name=f"random(n={n},acc={k},up={up},cycle={cycle})")


CASES = [graph(n, k, up, n + k, cycle)
         for n, k, up, cycle in ((1, 1, True, False), (2, 1, False, False), (33, 2, True, False), (64, 4, False, False),
                                 (511, 31, True, False), (512, 32, False, False), (513, 33, True, True),
                                 (4096, 255, True, False), (4096, 256, False, False), (4097, 257, False, True),
                                 (8191, 3, True, False), (8193, 0, False, False), (20000, 1200, False, False),
                                 (20001, 1251, True, False), (70001, 90, False, False), (70001, 30000, True, False))]


@pytest.mark.parametrize("direction", [False, True], ids=["pull", "direction-switch"])
@pytest.mark.parametrize("g", CASES, ids=lambda g: g.name)
def test_filtered_sweeps(mc, g, direction):
    csr = mc.build_csr(g.n, g.src, g.dst, transposed=direction)
    flags = mc.MAP_FLAG_STREAM | (mc.MAP_FLAG_DIRECTION if direction else 0)
    check_detect(mc, g, csr, flags=flags)
    check_detect(mc, g, csr, flags=flags, max_iterations=1, trace_cap=1)
    check_propagate_all(mc, g, csr, max_k=2, flags=flags)


def uniform(n, up, wrong=0, acc=0.002, seed=0):
    """Vertex v >= 2 has 1..7 edges to lower ids (higher, mirrored, where up), so that most rows grow in the middle
    of a fixpoint; `wrong` edges more point the other way."""
    rng = np.random.default_rng(seed + n)
    deg = rng.integers(1, 8, n)
    deg[0] = 0
    src = np.repeat(np.arange(1, n + 1, dtype=np.int64), deg)
    dst = 1 + rng.integers(0, 1 << 62, src.size) % (src - 1)
    if wrong:
        i = rng.choice(src.size, wrong, replace=False)
        src, dst = np.concatenate([src, dst[i]]), np.concatenate([dst, np.minimum(n, dst[i] + 1 + i % 1000)])
    if up:
        src, dst = n + 1 - src, n + 1 - dst
    a = np.zeros(n, np.uint8)
    a[rng.choice(n, int(acc * n), replace=False)] = 1
    return synth.Graph(n=n, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=a,
                       name=f"uniform(n={n},up={up},wrong={wrong})")


# From 2^20 vertices, edges one way (up to 1/64 of a sample the other): swept once in bands when the frontier is large.
@pytest.mark.parametrize("g", [uniform(1_100_003, False), uniform(1_048_576 + 4096, True), uniform(1_200_001, False, 3000),
                               uniform(1_200_033, True, 20000), uniform(1_100_000, False, 200_000)], ids=lambda g: g.name)
def test_banded_sweeps(mc, g):
    import oracle
    ref = oracle.map_detect(g, mode="desc")
    for flags in (mc.MAP_FLAG_DIRECTION, 0):
        csr = mc.build_csr(g.n, g.src, g.dst, transposed=flags != 0)
        check_detect(mc, g, csr, flags=flags, ref=ref)
    check_propagate_all(mc, g, csr, max_k=1)
