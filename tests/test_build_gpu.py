"""CSR builds at the edges of their paths: one workgroup in LDS (up to 12,288
vertices and 32,768 edges), one pass over a list that is sorted already, and
lists that only look sorted -- every row in edge-list order, byte for byte."""
import numpy as np
import pytest

from test_parity_gpu import _check_csr, mc  # noqa: F401

pytestmark = pytest.mark.gpu

SMALL = [(1, 0), (1, 1), (1, 40), (2, 63), (127, 64), (128, 1000), (129, 1025), (5000, 1023), (12288, 32768),
         (12288, 18431), (12289, 18432), (12288, 18433), (300, 18432), (4000, 30000), (3, 20000)]


def edges(n, m, seed, kind):
    rng = np.random.default_rng(seed)
    src = rng.integers(1, n + 1, m).astype(np.int32)
    dst = rng.integers(1, n + 1, m).astype(np.int32)
    if kind == "sorted":
        src = np.sort(src)
    if kind == "reverse":
        src = np.sort(src)[::-1].copy()
    if kind == "invalid" and m:
        bad = rng.choice(m, max(1, m // 50), replace=False)
        src[bad[::2]], dst[bad[1::2]] = n + 1, 0
        src[bad[:1]] = -2147483648
    return src, dst


@pytest.mark.parametrize("kind", ["random", "sorted", "reverse", "invalid"])
@pytest.mark.parametrize("n,m", SMALL)
def test_small_build(mc, n, m, kind):  # noqa: F811
    src, dst = edges(n, m, n * 7 + m, kind)
    csr = mc.build_csr(n, src, dst)
    assert int(csr.status.item()) == (mc.MAP_ERANGE_DEV if kind == "invalid" and m else 0)
    _check_csr(csr, n, src, dst)
    one = mc.build_csr(n, src, dst, transposed=False)
    _check_csr(one, n, src, dst, orientations=1)


@pytest.mark.parametrize("n,m", [(20000, 40001), (50, 300_003), (1 << 21, 1 << 20), (70000, (1 << 20) + 5)])
@pytest.mark.parametrize("case", ["sorted", "last edge out of order", "first edge out of order", "last edge invalid",
                                  "gaps"])
def test_sorted_list(mc, n, m, case):  # noqa: F811
    src, dst = edges(n, m, n + m, "sorted")
    if case == "gaps":   # no edge at the first and last rows
        src = np.clip(src, n // 4 + 1, n // 2 + 1)
    if case == "last edge out of order":
        src[-1] = 1
    if case == "first edge out of order":
        src[0] = n
    if case == "last edge invalid":
        dst[-1] = n + 1
    csr = mc.build_csr(n, src, dst)
    assert int(csr.status.item()) == (mc.MAP_ERANGE_DEV if case == "last edge invalid" else 0)
    _check_csr(csr, n, src, dst)


@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("m", [1000, 200_001])
def test_arrays_off_sixteen_bytes(mc, shift, m):  # noqa: F811
    import torch
    n = 30000
    src, dst = edges(n, m, m + shift, "sorted")
    s = torch.zeros(m + 8, dtype=torch.int32, device="cuda")[shift:shift + m]
    d = torch.zeros(m + 8, dtype=torch.int32, device="cuda")[shift:shift + m]
    s.copy_(torch.from_numpy(src))
    d.copy_(torch.from_numpy(dst))
    csr = mc.build_csr(n, s, d)
    assert int(csr.status.item()) == 0
    _check_csr(csr, n, src, dst)
