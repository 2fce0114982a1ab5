"""Windowed iterations that turn out short: two windows in a row of fewer than
four iterations or one of a single one (three in a row once one has paid) send
the run back to plain sweeps, and plain sweeps lead to windows again; windows
whose different records do not fit one list; one workspace shared by graphs
that enter windows.  Bit-exact against the CPU oracle.  A model of the rule by which windows are
entered, chosen and left, run on the oracle's removal sequence, asserts on the
CPU that each graph takes the route it is here for."""
import numpy as np
import pytest

import oracle
import synth
from test_parity_gpu import check_detect, mc  # noqa: F401

# As in the source: ids per window, ids that guide its choice, a strip that is small, accepting vertices needed,
# iterations of a window that paid, short ones in a row that end them (before and after one paid), plain iterations
# before the next try, records of the list.
BITS, FRONTS, FEW, LEFT, SHORT, SHORTS, BACKOFF, LIST = 224, 64, 28, 56, 4, (2, 3), 32, 8192


def strips(g):
    """Accepting sets A_1.. and removed ids of every iteration (None: it found a cycle or removed nothing)."""
    acc, dels, accs = g.acc.copy(), [], []
    while True:
        x, _ = oracle.fixpoint(g, acc, mode="desc")
        accs.append(acc)
        d = np.unique(x[x > 0])
        if d.size == 0 or (x == np.arange(1, g.n + 1)).any():
            return accs, dels + [None]
        dels.append(d)
        acc = acc.copy()
        acc[d - 1] = 0
        if not acc.any():
            return accs + [acc], dels


def window_ids(accepting, last):
    """The window that follows the strip `last`: equally many ids below each of its ids, BITS at most."""
    alive = np.flatnonzero(accepting)[::-1] + 1
    first = np.array([0]) if last.size > FRONTS else np.unique([np.count_nonzero(alive > x) for x in last])
    gap = np.maximum(np.append(first[1:], alive.size) - first, 0)
    each = max(d for d in range(alive.size + 1) if np.minimum(d, gap).sum() <= BITS)
    return {int(x) for p, n in zip(first, np.minimum(each, gap)) for x in alive[p:p + n]}


def route(g):
    """(iterations, [(iteration before the first window, that window's ids and accepting set, window lengths, back to
    plain)])."""
    accs, dels = strips(g)
    size = [d.size if d is not None else 1 << 30 for d in dels]
    out, k, again, backoff, seen = [], 0, 0, 0, 0
    while k < len(dels):
        k += 1
        seen += 1
        if dels[k - 1] is None or not (seen >= 3 and k >= again and size[k - 2] <= FEW and size[k - 3] <= FEW and
                                       accs[k - 1].sum() >= LEFT):
            continue
        entry, lengths, ids0, shorts, paid = k, [], None, 0, False
        while k < len(dels) and shorts < SHORTS[paid]:
            ids = window_ids(accs[k], dels[k - 1])
            ids0 = ids0 or (ids, accs[k])
            left, n = set(ids), 0
            while k < len(dels):
                k, n = k + 1, n + 1
                if dels[k - 1] is None:
                    break
                gone = set(dels[k - 1].tolist())
                left -= gone
                if not gone <= ids or not left:
                    break
            lengths.append(n)
            shorts = shorts + (SHORTS[0] if n == 1 and not paid else 1) if n < SHORT else 0
            paid = paid or n >= SHORT
        back = shorts >= SHORTS[paid] and k < len(dels) and dels[k - 1] is not None
        out.append((entry, ids0, lengths, back))
        if not back:
            break
        backoff = max(BACKOFF, 2 * backoff)
        again, seen = k + backoff, 0
    return len(dels), out


def scrambled(n, paths, k, seed, cycle=False):
    """Paths through k accepting vertices in random order of ids: an iteration strips the ids that no later vertex
    of the path exceeds, a few ids anywhere.  `cycle`: the start of a path is its own successor too."""
    rng = np.random.default_rng(seed)
    ids = rng.choice(n, k, replace=False).astype(np.int32) + 1
    parts = np.array_split(ids, paths)
    src, dst = np.concatenate([p[:-1] for p in parts]), np.concatenate([p[1:] for p in parts])
    if cycle:
        src, dst = np.append(src, ids[:1]), np.append(dst, ids[:1])
    acc = np.zeros(n, np.uint8)
    acc[ids - 1] = 1
    return synth.Graph(n=n, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=acc,
                       name=f"scrambled(n={n},paths={paths},accepting={k},cycle={cycle})")


def fan(k, chain):
    """k vertices that reach an accepting vertex of their own each and one chain of `chain` accepting vertices with
    larger ids: one id is stripped per iteration, and k different records remain."""
    v = np.arange(1, k + 1)
    c = 2 * k + 1 + np.arange(chain)
    src = np.concatenate([v, v, c[:-1]])
    dst = np.concatenate([v + k, np.full(k, c[0]), c[1:]])
    acc = np.zeros(2 * k + chain, np.uint8)
    acc[k:] = 1
    return synth.Graph(n=2 * k + chain, src=src.astype(np.int32), dst=dst.astype(np.int32), acc=acc,
                       name=f"fan({k},{chain})")


def records(g, ids, accepting):
    """Different records (window ids reached, largest other accepting id reached) of a graph whose edges ascend."""
    bit = {x: 1 << i for i, x in enumerate(sorted(ids))}
    mask, low = [0] * (g.n + 1), [0] * (g.n + 1)
    succ = [[] for _ in range(g.n + 1)]
    for s, d in zip(g.src.tolist(), g.dst.tolist()):
        assert s < d
        succ[s].append(d)
    for v in range(g.n, 0, -1):
        for w in succ[v]:
            mask[v] |= mask[w] | bit.get(w, 0)
            low[v] = max(low[v], low[w], w if accepting[w - 1] and w not in bit else 0)
    return len(set(zip(mask[1:], low[1:])))


RETURNS = [scrambled(13000, 1, 900, 2), scrambled(20011, 1, 1500, 1), scrambled(40000, 1, 3000, 1),
           scrambled(13000, 1, 900, 1, cycle=True), scrambled(13000, 1, 1500, 2, cycle=True), scrambled(16384, 2, 1100, 4)]
OVERFLOW = [fan(10000, 120), fan(12000, 200)]


@pytest.mark.parametrize("g", RETURNS, ids=lambda g: g.name)
def test_route_goes_back_and_forth(g):
    _, r = route(g)
    assert len(r) >= 2 and r[0][3], [x[2:] for x in r]


@pytest.mark.parametrize("g", OVERFLOW, ids=lambda g: g.name)
def test_route_overflows_the_list(g):
    k, r = route(g)
    assert len(r) == 1 and r[0][0] == 3 and r[0][2][0] >= SHORT
    assert records(g, *r[0][1]) > LIST


@pytest.mark.gpu
@pytest.mark.parametrize("g", RETURNS + OVERFLOW, ids=lambda g: g.name)
def test_returns_and_overflows(mc, g):  # noqa: F811
    csr = mc.build_csr(g.n, g.src, g.dst)
    _, ref = check_detect(mc, g, csr)
    check_detect(mc, g, csr, flags=mc.MAP_FLAG_NO_TRACE_DIGEST, trace_cap=7, ref=ref)


@pytest.mark.gpu
@pytest.mark.parametrize("cap", [3, 4, 5, 6, 7, *range(35, 42), 50, 51, 52])
def test_capped_around_a_return(mc, cap):  # noqa: F811
    check_detect(mc, RETURNS[0], max_iterations=cap)


@pytest.mark.gpu
def test_shared_workspace(mc):  # noqa: F811
    """Graphs of different sizes that enter windows, a plain run between them, twice on one workspace."""
    graphs = [RETURNS[0], synth.config2(seed=22, n=32768, planted=True), synth.config1(n=30000, dag=True), OVERFLOW[0],
              RETURNS[1]]
    ws = mc.workspace(max(g.n for g in graphs), max(g.m for g in graphs))
    refs = [oracle.map_detect(g, mode="desc") for g in graphs]
    csrs = [mc.build_csr(g.n, g.src, g.dst) for g in graphs]
    for _ in range(2):
        for g, csr, ref in zip(graphs, csrs, refs):
            out = mc.detect(csr, g.acc, trace_cap=g.n_acc + 1, want_acc=True, ws=ws)
            assert out.result.status == 0 and out.result.verdict == ref.verdict, g.name
            assert np.array_equal(out.accepting_out, ref.acc_out), g.name
            assert np.array_equal(out.trace[:, [0, 2]], ref.trace[:out.trace.shape[0], [0, 2]]), g.name
