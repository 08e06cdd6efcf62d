"""Unweighting with the terms of 64 trials shared by a workgroup's wavefronts
(8 terms each, 1 to 8 wavefronts): channels and peaks without a channel at and
beside whole shares and rounds of shares, batches beside whole groups of 64
trials and at the sizes where fewer wavefronts share, against the oracle's
decisions from the same state."""
import numpy as np
import pytest

import workloads as W
from gpu_util import pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,K,orphans,batch", [
    (2, 1, 0, 63), (3, 8, 0, 65), (3, 9, 0, 1000), (4, 33, 0, 65_536), (5, 65, 3, 700),
    (4, 30, 4, 65_600), (3, 20, 0, 131_072), (2, 4, 1, 300_000),
])
def test_shared_terms_parity(d, K, orphans, batch):
    p = W.gauss_mixture(d, K + orphans, 20, 11 + K)
    if orphans:
        p = p.with_(chan_kind=p.chan_kind[:K], chan_loc=p.chan_loc[:K], chan_width=p.chan_width[:K])
    gpu, orc = pair(p)
    N = 50_000
    for _ in range(2):
        gpu.sample_iteration(N)
        orc.sample_iteration(N, 8)
        gpu.refine()
        orc.refine()
    gpu.sample_iteration(N)
    orc.sample_iteration(N, 8)
    orc.edges = gpu.edges  # identical state, as the maximum weight
    orc.wmax = gpu.history[-1, 3]
    n_ev = 300
    ev_g, st_g = gpu.unweight(n_ev, batch=batch)
    ev_o, st_o = orc.unweight(n_ev, batch=batch)
    assert st_o["accept_ties"] == 0
    assert st_g["trials"] == st_o["trials"]
    assert st_g["w_max"] == pytest.approx(st_o["w_max"], rel=1e-12)
    assert np.max(np.abs(ev_g.cpu().numpy() - ev_o)) < 1e-12
