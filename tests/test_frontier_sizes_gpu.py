"""Counterexample and pruning where the frontiers begin to be staged (8 workgroups,
one per 4,096 vertices), against the CPU oracle."""
import numpy as np
import pytest

import oracle
import synth
from test_parity_gpu import mc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4096, 28_672, 28_673, 32_769, 40_000])
def test_few_and_many_workgroups(mc, n):  # noqa: F811
    for g in (synth.config2(seed=n, n=n, planted=True), synth.random_graph(n, n, 2 * n, p_acc=0.05)):
        csr = mc.build_csr(g.n, g.src, g.dst)
        keep, acc = oracle.trim(g)
        out = mc.trim(csr, g.acc)
        assert out.status == 0 and out.kept == int(keep.sum()) and out.accepting_kept == int(acc.sum()), g.name
        assert np.array_equal(out.keep.cpu().numpy(), keep) and np.array_equal(out.accepting.cpu().numpy(), acc)
        for w in (g.planted[0] if len(g.planted) else n // 2, n // 3):
            got, ref = mc.lasso(csr, int(w), 1), oracle.lasso(g, int(w), 1)
            assert (got.stem_len, got.cycle_len) == (ref.stem_len, ref.cycle_len), (g.name, w, got)
            if ref.path is not None:
                assert got.status == 0 and np.array_equal(got.path, ref.path), (g.name, w)


@pytest.mark.parametrize("leaves", [8191, 8192, 8193])
def test_stage_filled_by_one_wave(mc, leaves):  # noqa: F811
    """1 -> every leaf -> w -> 1 among enough vertices that the frontiers are staged."""
    n, w = 40_000, leaves + 2
    leaf = np.arange(2, w, dtype=np.int32)
    src = np.concatenate([np.full(leaves, 1), leaf, [w]]).astype(np.int32)
    dst = np.concatenate([leaf, np.full(leaves, w), [1]]).astype(np.int32)
    acc = np.zeros(n, np.uint8)
    acc[w - 1] = 1
    for cut in (0, 1):   # without the edge back to 1 everything is removed
        g = synth.Graph(n=n, src=src[:src.size - cut].copy(), dst=dst[:dst.size - cut].copy(), acc=acc, name="star")
        csr = mc.build_csr(g.n, g.src, g.dst)
        keep, _ = oracle.trim(g)
        out = mc.trim(csr, g.acc)
        assert out.status == 0 and np.array_equal(out.keep.cpu().numpy(), keep)
        got, ref = mc.lasso(csr, w, 1), oracle.lasso(g, w, 1)
        assert (got.stem_len, got.cycle_len) == (ref.stem_len, ref.cycle_len)
        if ref.path is not None:
            assert np.array_equal(got.path, ref.path)
