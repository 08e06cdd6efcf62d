"""A new job's history is empty whatever its length: the workgroups that clear
it at their edges (512 rows each, at most 1024 of them), with memory of an
earlier job's history handed back by the allocator."""
import numpy as np
import pytest

import workloads as W
from gpu_util import mcv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 511, 512, 513, 1000, 65_536, 600_001])
def test_history_starts_empty(rows):
    p = W.gauss_mixture(2, 1, 5, 3)
    M = mcv()
    gpu = M.Integrator(p, max_iterations=rows)
    blob = np.frombuffer(gpu.save_state(), np.uint8).copy()
    head, edges, alpha = 16 * 8, 1 * 2 * 6 * 8, 8
    history = slice(head + edges + alpha, head + edges + alpha + rows * 5 * 8)
    assert not blob[history].any()
    # leave other values behind, as a saved state's, and start anew
    blob[history] = np.ones(rows * 5).view(np.uint8)
    gpu.load_state(blob.tobytes())
    gpu.close()
    again = M.Integrator(p, max_iterations=rows)
    assert not np.frombuffer(again.save_state(), np.uint8)[history].any()
    again.close()
