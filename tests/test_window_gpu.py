"""Windowed iterations (graphs of more than 12,288 vertices whose strips remove
few flags each) against the CPU oracle, bit-exact: every iteration's removals
and digest, verdict, accepting set, capped runs, runs that leave the windows
and come back."""
import numpy as np
import pytest

import synth
from test_parity_gpu import check_detect, mc  # noqa: F401

pytestmark = pytest.mark.gpu


def chains(n, parts, every, up=True, shuffle_seed=None, cycle_at=None, back=0):
    """`parts` disjoint chains over consecutive ids, every `every`-th vertex accepting: one strip per chain and
    iteration.  `back`: extra edges to lower vertices between two accepting ones; `cycle_at`: a vertex with a
    back edge over itself (an accepting cycle)."""
    v = np.arange(1, n, dtype=np.int32)
    edges = v % max(1, n // parts) != 0
    src, dst = v[edges], v[edges] + 1
    if not up:
        src, dst = dst, src
    acc = np.zeros(n, np.uint8)
    acc[every - 1::every] = 1
    rng = np.random.default_rng(n + parts)
    if back:
        s = rng.integers(2, n, back).astype(np.int32)
        s = s[(s % every > 1)]
        src, dst = np.concatenate([src, s]), np.concatenate([dst, s - 1])
    if cycle_at:
        a = (cycle_at // every) * every
        src, dst = np.append(src, np.int32(a + 1)), np.append(dst, np.int32(a))
        if not up:
            src, dst = np.append(src, np.int32(a)), np.append(dst, np.int32(a + 1))
    if shuffle_seed is not None:
        o = np.random.default_rng(shuffle_seed).permutation(src.size)
        src, dst = src[o], dst[o]
    return synth.Graph(n=n, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=acc,
                       name=f"chains(n={n},parts={parts},every={every},up={up},cycle={cycle_at},back={back})")


def sparse_accepting(seed, n, m, k):
    g = synth.random_graph(seed, n, m, p_acc=0.0)
    acc = np.zeros(n, np.uint8)
    acc[np.random.default_rng(seed).choice(n, k, replace=False)] = 1
    src, dst = np.minimum(g.src, g.dst), np.maximum(g.src, g.dst)
    keep = src != dst
    return synth.Graph(n=n, src=src[keep].copy(), dst=dst[keep].copy(), acc=acc, name=f"upward(n={n},m={m},acc={k})")


def hub_states(n, deg):
    """A state space with one vertex of `deg` successors in its own block and one of `deg` anywhere."""
    g = synth.config2(seed=8, n=n)
    src = np.concatenate([g.src, np.full(deg, 5, np.int32), np.full(deg, 9, np.int32)])
    dst = np.concatenate([g.dst, 6 + np.arange(deg, dtype=np.int32) % 900,
                          np.random.default_rng(3).integers(10, n + 1, deg).astype(np.int32)])
    return synth.Graph(n=n, src=src, dst=dst, acc=g.acc, name=f"hub-states(n={n},deg={deg})")


CASES = [
    chains(12289, 1, 40), chains(13000, 1, 25, up=False), chains(20000, 7, 50, back=300),
    chains(20000, 20, 60, shuffle_seed=1), chains(30000, 3, 100, up=False, back=500, shuffle_seed=2),
    chains(20011, 2, 40, cycle_at=6000), chains(20011, 1, 40, up=False, cycle_at=15000),
    sparse_accepting(5, 15000, 40000, 400), sparse_accepting(6, 40000, 60000, 800),
    synth.config2(seed=21, n=12300), synth.config2(seed=22, n=32768, planted=True), synth.config2(seed=23, n=70001),
    synth.config2(seed=24, n=200003, planted=True), hub_states(20000, 3000), hub_states(16384, 30000),
]


@pytest.mark.parametrize("g", CASES, ids=lambda g: g.name)
def test_windowed_iterations(mc, g):  # noqa: F811
    csr = mc.build_csr(g.n, g.src, g.dst)
    out, ref = check_detect(mc, g, csr)
    check_detect(mc, g, csr, flags=mc.MAP_FLAG_NO_TRACE_DIGEST, trace_cap=min(ref.iterations, 7), ref=ref)


@pytest.mark.parametrize("cap", [3, 4, 5, 6, 20, 41, 62, 63])
def test_capped_inside_a_window(mc, cap):  # noqa: F811
    g = synth.config2(seed=6, n=50001)   # 62 iterations
    check_detect(mc, g, max_iterations=cap)


def test_same_workspace_twice(mc):  # noqa: F811
    """Words that a windowed run leaves in the workspace mean nothing to the next run on it."""
    a, b = synth.config2(seed=22, n=32768, planted=True), synth.config1(n=30000, dag=True)
    ws = mc.workspace(a.n, max(a.m, b.m))
    ca, cb = mc.build_csr(a.n, a.src, a.dst), mc.build_csr(b.n, b.src, b.dst)
    first = [mc.detect(ca, a.acc, ws=ws).result.verdict, mc.detect(cb, b.acc, ws=ws).result.verdict]
    again = [mc.detect(ca, a.acc, ws=ws).result.verdict, mc.detect(cb, b.acc, ws=ws).result.verdict]
    assert first == again
    check_detect(mc, a, ca)
    check_detect(mc, b, cb)
