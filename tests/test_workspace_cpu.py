"""The bytes of a workspace never fall as a graph grows, so that one workspace
for the largest n and the largest m of a set serves every graph of it."""
import itertools

import paper_0912_2555_amd as mc

N = sorted({1, 2, 300, 1 << 22, 1 << 25, (1 << 31) - 2} |
           {b + d for b in (1024, 4096, 12_288, 1 << 16, 1 << 20, 1 << 24) for d in (-257, -1, 0, 1, 256)})
M = sorted({0, 1, 64, 5000, 1 << 24, (1 << 31) - 1} |
           {b + d for b in (4096, 18_432, 49_152, 1 << 20) for d in (-1, 0, 1)})


def test_workspace_bytes_never_fall():
    got = {(n, m): mc.map_workspace_bytes(n, m) for n in N for m in M}
    assert all(got.values())
    for (a, b), m in itertools.product(zip(N, N[1:]), M):
        assert got[a, m] <= got[b, m], (a, b, m)
    for n, (a, b) in itertools.product(N, zip(M, M[1:])):
        assert got[n, a] <= got[n, b], (n, a, b)


def test_job_and_batch_bytes_never_fall():
    for (a, b), m in itertools.product(zip(N, N[1:]), M):
        assert mc.map_job_scratch_bytes(a, m) <= mc.map_job_scratch_bytes(b, m), (a, b, m)
    for a, b in zip(N, N[1:]):
        assert mc.map_batch_workspace_bytes(1, a) <= mc.map_batch_workspace_bytes(1, b), (a, b)
