"""Point selection where one pass over the orbitals forms several columns
(orbitals above 20 MB): every pivot against the oracle's greedy selector."""
import dataclasses

import numpy as np
import pytest

import isdf_inputs as inp
from oracle import ipselect as ips

pytestmark = pytest.mark.gpu


# 2520 grid points: 39.4 blocks of 64 (a block's maximum is a candidate for the
# pass) and 4.9 of 512; 4096: whole ones.  576, 625 and 375 rows: row slices whole
# and ragged.  200 pivots are many refills of the held columns.
@pytest.mark.parametrize("grid,kmesh,n_orb", [((12, 15, 14), (4, 4, 4), 9), ((14, 15, 12), (5, 5, 5), 5),
                                             ((16, 16, 16), (3, 5, 5), 5)])
@pytest.mark.parametrize("device", [False, True])
def test_every_pivot_equals_oracle(grid, kmesh, n_orb, device):
    import torch
    import paper_2601_16379_amd as pkg
    n = 200
    cfg = dataclasses.replace(inp.get_config("t_mid_k4"), grid=grid, kmesh=kmesh, n_orb=n_orb, n_ip=n)
    d = inp.make_inputs(cfg)
    assert d.orbitals.nbytes > 20 << 20
    orb = torch.from_numpy(d.orbitals).cuda() if device else d.orbitals
    ip, res = pkg.select_points(cfg.grid, cfg.kmesh, orb, n)
    piv, dmax, _, _, gap = ips.pivoted_cholesky_points(d.orbitals, n, with_gaps=True)
    # a choice closer than this to the runner-up is a matter of rounding
    assert gap.min() > 1e-9 * dmax[0]
    bad = np.nonzero(np.asarray(ip) != piv)[0]
    assert bad.size == 0, "first differing pivot at step %d" % bad[0]
    assert np.max(np.abs(res - dmax)) < 1e-10 * dmax[0]
