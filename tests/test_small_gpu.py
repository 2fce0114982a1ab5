"""One-workgroup detection of graphs of up to 12,288 vertices: the edges of its
ranges against the CPU oracle, bit-exact (verdict, K, removals, digests,
accepting set, map vectors), alone and as members of a batch."""
import numpy as np
import pytest

import oracle
import synth
from test_parity_gpu import check_detect, check_propagate_all, mc  # noqa: F401

pytestmark = pytest.mark.gpu

N, EDGES = 12288, 49152   # vertices in LDS, edges in registers


def hub(n, deg, seed):
    """A sparse random digraph with two rows of `deg` edges."""
    g = synth.random_graph(seed, n, 2 * n, p_acc=0.05)
    rng = np.random.default_rng(seed)
    src = np.concatenate([g.src, np.repeat(np.array([n // 2, n], np.int32), deg)])
    dst = np.concatenate([g.dst, rng.integers(1, n + 1, 2 * deg).astype(np.int32)])
    return synth.Graph(n=n, src=src, dst=dst, acc=g.acc, name=f"hub(n={n},deg={deg})")


def ladder(n, up):
    """Long chains of accepting vertices: many outer iterations, values going up or down the rows."""
    v = np.arange(1, n, dtype=np.int32)
    acc = np.zeros(n, np.uint8)
    acc[::7] = 1
    src, dst = (v, v + 1) if up else (v + 1, v)
    return synth.Graph(n=n, src=src.copy(), dst=dst.copy(), acc=acc, name=f"chain(n={n},up={up})")


CASES = [
    *[synth.random_graph(40 + i, n, int(1.3 * n) + 1, p_acc=0.1) for i, n in
      enumerate([1, 2, 64, 1023, 1024, 1025, 2049, N - 1, N, N + 1])],
    *[synth.random_graph(60 + i, N, m, p_acc=0.02) for i, m in enumerate([0, 1023, 8193, EDGES - 1, EDGES, EDGES + 1])],
    hub(300, 65, 1), hub(5000, 513, 2), hub(4000, 60000, 3), ladder(300, True), ladder(300, False),
    synth.config1(n=9001, dag=True), synth.config2(seed=5, n=9001, planted=True),
    synth.config1(n=3000, dag=False), synth.random_graph(9, 70, 6000, p_acc=0.5),
]


@pytest.mark.parametrize("g", CASES, ids=lambda g: f"{g.name}-{g.m}")
def test_small_graph(mc, g):  # noqa: F811
    csr = mc.build_csr(g.n, g.src, g.dst)
    check_detect(mc, g, csr)
    check_detect(mc, g, csr, max_iterations=1, trace_cap=1)
    check_propagate_all(mc, g, csr, max_k=3)


def test_small_graphs_in_a_batch(mc):  # noqa: F811
    csrs = [mc.build_csr(g.n, g.src, g.dst) for g in CASES]
    b = mc.Batch(csrs, [g.acc for g in CASES])
    b.launch()
    for g, r in zip(CASES, b.read()):
        ref = oracle.map_detect(g, mode="desc")
        assert r.status == 0 and r.verdict == ref.verdict and r.accepting_left == ref.accepting_left, g.name
