"""Frontiers around the size a workgroup stages (8,192 entries), in the counterexample search and the pruning,
against the CPU oracle: all vertices at once, and one vertex whose expansion by a single wave fills the stage."""
import numpy as np
import pytest

import synth
from test_lasso_gpu import check, mc  # noqa: F401
from test_trim_gpu import check_trim

pytestmark = pytest.mark.gpu


def star(leaves):
    """1 -> every leaf -> w -> 1: the search's second frontier is every leaf."""
    w = leaves + 2
    leaf = np.arange(2, w, dtype=np.int32)
    src = np.concatenate([np.full(leaves, 1, np.int32), leaf, [w]]).astype(np.int32)
    dst = np.concatenate([leaf, np.full(leaves, w, np.int32), [1]]).astype(np.int32)
    acc = np.zeros(w, np.uint8)
    acc[w - 1] = 1
    return synth.Graph(n=w, src=src, dst=dst, acc=acc, name=f"star({leaves})")


@pytest.mark.parametrize("leaves", [1, 8191, 8192, 8193, 30000])
def test_search_and_pruning_through_a_star(mc, leaves):
    g = star(leaves)
    csr = mc.build_csr(g.n, g.src, g.dst)
    check(mc, g, csr, g.n, 1)
    check_trim(mc, g)
    # Without the edge back to 1 the leaves are removed one round after it.
    check_trim(mc, synth.Graph(n=g.n, src=g.src[:-1].copy(), dst=g.dst[:-1].copy(), acc=g.acc, name=g.name + "-open"))


@pytest.mark.parametrize("n", [1024, 1025, 2_097_152, 2_300_001])
def test_pruning_of_a_graph_without_cycles_in_one_round(mc, n):
    acc = np.ones(n, np.uint8)
    check_trim(mc, synth.Graph(n=n, src=np.array([1], np.int32), dst=np.array([n], np.int32), acc=acc, name=f"edge({n})"))
