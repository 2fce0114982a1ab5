"""CSR builds of ascending lists that leave long runs of vertices without an
edge -- before the first edge, between two and after the last, a few edges over
many vertices -- and of lists that ascend in pieces only, byte for byte."""
import numpy as np
import pytest

from test_parity_gpu import _check_csr, mc  # noqa: F401

pytestmark = pytest.mark.gpu


def teeth(n, m, length):
    """Ascending pieces of `length` edges over all vertices.  The 1,024 evenly
    spaced pairs of neighbours by which a list is taken as ascending ascend."""
    pairs = set(((m - 1) * np.arange(1024, dtype=np.int64) // 1024).tolist())
    step = n // (2 * length)
    key, at = np.empty(m, np.int32), 0
    for i in range(m):
        at = 0 if at >= length and i - 1 not in pairs else at
        key[i] = min(1 + step * at, n)
        at += 1
    return key


KEYS = {
    "few": lambda n, m, rng: np.sort(rng.integers(1, n + 1, m)),
    "late": lambda n, m, rng: np.sort(rng.integers(n - n // 50, n + 1, m)),
    "early": lambda n, m, rng: np.sort(rng.integers(1, n // 50 + 2, m)),
    "split": lambda n, m, rng: np.sort(np.where(rng.random(m) < 0.5, rng.integers(1, n // 50 + 2, m),
                                                rng.integers(n - n // 50, n + 1, m))),
    "last": lambda n, m, rng: np.full(m, n),
    "edge": lambda n, m, rng: np.sort(np.minimum(1 + 512 * rng.integers(0, n // 512, m) + rng.integers(0, 3, m), n)),
    "teeth": lambda n, m, rng: teeth(n, m, 16),
}


@pytest.mark.parametrize("kind", sorted(KEYS))
@pytest.mark.parametrize("n,m", [(12289, 3), (20000, 1), (20000, 40000), (300001, 257), (1000003, 300), (3000000, 50001),
                                 (400000, 1200001)])
def test_long_gaps(mc, n, m, kind):  # noqa: F811
    rng = np.random.default_rng(n + m)
    src = KEYS[kind](n, m, rng).astype(np.int32)
    dst = rng.integers(1, n + 1, m).astype(np.int32)
    csr = mc.build_csr(n, src, dst)
    assert int(csr.status.item()) == 0
    _check_csr(csr, n, src, dst)
