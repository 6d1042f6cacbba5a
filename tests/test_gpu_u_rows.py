"""bf16x3 U^q where the pair rows lie 4 MB and more apart (504 classes, about a
thousand points), which runs two workgroups a CU: fragment ERIs against the FP64
path within the mixed bar of 1e-6 Eh, with the factor of W^q (column tiles of
differing length, in turned and in plain order) and without."""
import dataclasses

import numpy as np
import pytest

import isdf_inputs as inp

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n_ip", [977, 1040, 1100])    # 8 column tiles (turned order), a strip of 16, 76 columns
@pytest.mark.parametrize("plain", [False, True])
def test_rows_far_apart(n_ip, plain):
    import torch
    import paper_2601_16379_amd as pkg
    cfg = dataclasses.replace(inp.get_config("t_mid_k4"), kmesh=(10, 10, 10), n_orb=6, n_ip=n_ip)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, torch.from_numpy(d.orbitals).cuda(),
                   torch.from_numpy(d.ip_index).cuda(), w_plain=plain)
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    assert ctx.stats()["w_factor"] is not plain
    # 1, 49, 121 and 400 pair rows: below, at and above the 32-row strips and 128-row tiles
    frags = [torch.from_numpy(inp.make_fragment(cfg, f, n)).cuda() for f, n in enumerate((1, 7, 11, 20))]
    ref = ctx.fragment_eri(frags, "fp64")
    out = ctx.fragment_eri(frags, "bf16x3")
    one = ctx.fragment_eri(frags[3:], "bf16x3", pair_blocks=3)[0]
    for a, b in zip(out, ref):
        assert float((a - b).abs().max()) < 1e-6
        assert float((a - b).abs().max()) < 1e-4 * float(b.abs().max())
    assert torch.equal(one, out[3])               # blocked: the same products in other tiles
    ctx.close()
