"""Dense graphs of up to 12,288 vertices at the edges of the rule that gives them
to one workgroup or to several, with workspaces that bound the edges, that do
not, and without one: bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from test_parity_gpu import mc  # noqa: F401

pytestmark = pytest.mark.gpu

LIMIT = 3 << 18   # edges that one workgroup takes from several


def dense(n, m):
    """Edges to lower ids, sorted by source; a few accepting vertices."""
    rng = np.random.default_rng(n + m)
    a = rng.integers(2, n + 1, m)
    src, dst = np.sort(a).astype(np.int32), None
    dst = (rng.integers(0, 1 << 30, m) % (src - 1) + 1).astype(np.int32)
    acc = np.zeros(n, np.uint8)
    acc[rng.choice(n, max(1, n // 50), replace=False)] = 1
    return synth.Graph(n=n, src=src, dst=dst, acc=acc, name=f"dense(n={n},m={m})")


CASES = [(2048, LIMIT + 1), (2049, LIMIT), (2049, LIMIT + 1), (4096, 2 << 20), (4096, (2 << 20) + 1), (4097, 3 << 20),
         (6144, (3 << 20) + 1), (6145, (4 << 20) + 1), (12288, LIMIT), (12288, LIMIT + 1), (12289, LIMIT + 1),
         (12288, 20000)]


@pytest.mark.parametrize("n,m", CASES)
def test_dense_graph(mc, n, m):  # noqa: F811
    import torch
    g = dense(n, m)
    ref = oracle.map_detect(g, mode="desc")
    want, _ = oracle.fixpoint(g, mode="desc")
    csr = mc.build_csr(n, g.src, g.dst, transposed=False)
    acc = torch.from_numpy(g.acc).cuda()
    cap = g.n_acc + 1
    for space in ("exact", "large", "smallest", "none"):
        ws = mc.workspace(n, {"exact": m, "large": 8 * m, "smallest": 0, "none": 0}[space])
        res, trace = mc.new_result(), torch.zeros((cap, 3), dtype=torch.int64, device="cuda")
        out = torch.zeros(n, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            res.fill_(-7)
            if space == "none":
                rc = mc.map_detect_noalloc(n, csr.row_ptr, csr.col, acc, res, trace, out, 0, 0)
            else:
                rc = mc.map_detect(n, csr.row_ptr, csr.col, None, None, acc, res, trace, out, 0, 0, ws)
            assert rc == 0
            r = mc.Result.from_tensor(res)
            assert r.status == 0 and r.verdict == ref.verdict and r.accepting_left == ref.accepting_left, (space, r)
            assert np.array_equal(out.cpu().numpy(), ref.acc_out)
            t = trace.cpu().numpy().view(np.uint64)[:r.iterations]
            assert np.array_equal(t[:, [0, 2]], ref.trace[:, [0, 2]])
        if space != "none":
            got = torch.full((n,), -1, dtype=torch.int32, device="cuda")
            assert mc.map_propagate(n, csr.row_ptr, csr.col, None, None, acc, got, res, 0, ws) == 0
            assert np.array_equal(got.cpu().numpy(), want)


def test_named_workspace_bytes(mc):  # noqa: F811
    """The wrappers name the graph's own share of a large workspace, and no more than there is."""
    import torch
    ws = torch.empty(mc.map_workspace_bytes(1 << 20, 1 << 22), dtype=torch.uint8, device="cuda")
    assert mc._loop_ws_bytes(ws, 5000, ws[:9000]) == mc.map_workspace_bytes(5000, 9000)
    assert mc._loop_ws_bytes(ws, 20000, ws[:9000]) == ws.numel()
    small = ws[:mc.map_workspace_bytes(5000, 9000)]
    assert mc._loop_ws_bytes(small, 5000, ws[:2000]) == small.numel() and mc._loop_ws_bytes(None, 5, None) == 0
