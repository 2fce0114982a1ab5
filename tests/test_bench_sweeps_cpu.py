"""bench.py credits no edge traffic to iterations that read no edge (CPU only)."""
import os
import sys

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_passes_over_records_are_no_sweeps_over_edges():
    # A plain iteration, a window of four iterations, a window that stripped an id outside it at once, a last iteration.
    trace = np.array([[8, 14, 0], [8, 11, 0], [9, 1, 0], [7, 1, 0], [8, 1, 0], [5, 9, 0], [0, 2, 0]], np.int64)
    assert bench.edge_sweeps(trace) == 14 + 11 + 9 + 2
    assert bench.edge_sweeps(trace.view(np.uint64)) == 36 and bench.edge_sweeps(np.zeros((1, 3), np.int64)) == 0
