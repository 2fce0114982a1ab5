"""Phase counters of the measurement build describe the last launch, also where
one workgroup solved a small graph."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = """
import numpy as np, paper_0912_2555_amd as mc, synth
from test_small_gpu import ladder
for g in (ladder(300, True), synth.random_graph(7, 900, 60000, p_acc=0.1)):
    out = mc.detect(mc.build_csr(g.n, g.src, g.dst), g.acc)
    ph = mc.phase_counters()
    assert ph.shape == (1, 16), ph.shape
    assert ph[0, 8] == out.result.sweeps and ph[0, 11] == out.result.iterations, (ph, out.result)
    assert ph[0, 0] > 0 and ph[0, 6] > 0 and (ph[0, 2] > 0) == (g.m <= 49152) and (ph[0, 3] > 0) == (g.m > 49152), ph
print("counters ok")
"""


def test_counters_of_a_small_graph():
    lib = os.path.join(ROOT, "paper_0912_2555_amd", "libmapcheck_phases.so")
    env = dict(os.environ, MAPCHECK_LIB=lib, PYTHONPATH=os.pathsep.join([ROOT, os.path.join(ROOT, "tests")]))
    r = subprocess.run([sys.executable, "-c", PROGRAM], capture_output=True, text=True, timeout=100, env=env, cwd=ROOT)
    assert r.returncode == 0 and "counters ok" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
