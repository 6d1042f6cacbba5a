"""Edges of the fragment products' tiles, against the oracle.

Given the GPU's own W^q, the fragment ERIs of eqs. (19)-(20) are products of
sizes N_IP and n_f^2: interpolation-point counts and fragment sizes one below,
at and one above the tile, strip and stage sizes (16, 32, 64, 128), with few
tiles (small tiles) and with many (large ones).  Bars: the repository's own,
1e-10 of the largest ERI in FP64 and 1e-6 Eh in FP32 and bf16x3."""
import dataclasses

import numpy as np
import pytest

import isdf_inputs as inp
from oracle import kpoint as ko

pytestmark = pytest.mark.gpu

FEW = [1, 2, 3, 4, 5, 6, 8, 9, 11]                # n_f^2 = 1 .. 121
MANY = [24, 25, 41, 46]                           # n_f^2 = 576 .. 2116: over a thousand 64 x 64 tiles


def _context(n_ip):
    import torch
    import paper_2601_16379_amd as pkg
    cfg = dataclasses.replace(inp.get_config("t_small_k2"), n_ip=n_ip)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, torch.from_numpy(d.orbitals).cuda(),
                   torch.from_numpy(d.ip_index).cuda())
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    return cfg, ctx, ko.ip_values(d.orbitals, d.ip_index), np.stack([ctx.get_kernel(q) for q in range(cfg.n_k)])


def _check(cfg, ctx, x, w, sizes, precs):
    import torch
    frags = [inp.make_fragment(cfg, f, n) for f, n in enumerate(sizes)]
    dev = [torch.from_numpy(f).cuda() for f in frags]
    out = {p: ctx.fragment_eri(dev, p) for p in precs}
    for f, c in enumerate(frags):
        ref = ko.fragment_eri(x, c, w, cfg.kmesh)
        big = np.max(np.abs(ref))
        for p in precs:
            err = np.max(np.abs(out[p][f].cpu().numpy() - ref))
            assert err <= (1e-10 * big if p == "fp64" else 1e-6), (sizes[f], p, err, big)


@pytest.mark.parametrize("n_ip", [15, 16, 17, 31, 33, 48, 63, 64, 65, 97, 127, 129])
def test_small_products(n_ip):
    cfg, ctx, x, w = _context(n_ip)
    _check(cfg, ctx, x, w, FEW, ["fp64", "fp32", "bf16x3"])
    ctx.close()


@pytest.mark.parametrize("n_ip", [72, 129])
def test_many_tiles(n_ip):
    cfg, ctx, x, w = _context(n_ip)
    _check(cfg, ctx, x, w, MANY, ["fp64", "fp32", "bf16x3"])
    ctx.close()


@pytest.mark.parametrize("n_ip", [8, 63, 64, 65, 72, 121, 127, 128, 129, 140])
def test_factor_edges(n_ip):
    """Blocked factor and inverse at block edges, complex metrics: Pi^q W^q
    Pi^q against the oracle's V^q (eq. (8)) within the first-order bound
    8 n u cond(Pi^q) of the two-sided solve."""
    import paper_2601_16379_amd as pkg
    cfg = dataclasses.replace(inp.get_config("t_small_k3"), n_ip=n_ip)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, d.orbitals, d.ip_index)
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    x = ko.ip_values(d.orbitals, d.ip_index)
    for q in (0, 1, 9):
        pi, w = ctx.get_metric(q), ctx.get_kernel(q)
        v = ko.coulomb_kernel_of(ko.rhs(x, d.orbitals, cfg.kmesh, [q])[0], d.lattice, cfg.grid, cfg.kmesh, q)
        ev = np.linalg.eigvalsh(pi)
        bound = 8 * n_ip * 2.0 ** -53 * ev[-1] / ev[0]
        err = np.max(np.abs(pi @ w @ pi - v)) / np.max(np.abs(v))
        assert ev[0] > 0 and err <= bound, (q, err, bound)
    ctx.close()


@pytest.mark.parametrize("kmesh", [(4, 2, 4), (4, 4, 3), (4, 3, 3), (3, 4, 2), (4, 1, 4), (6, 6, 6)])
@pytest.mark.parametrize("n_ip", [15, 33, 65])
def test_pair_transform_points(kmesh, n_ip):
    """The register pair transform with two lanes a point (four along axis 1
    and an even number, 8 or more, across) and one, and the line transform, at
    point counts one off their chunks (32, 64, 16); runs of q longer and
    shorter than a workgroup's waves."""
    import paper_2601_16379_amd as pkg
    cfg = dataclasses.replace(inp.get_config("t_small_k2"), kmesh=kmesh, n_ip=n_ip)
    d = inp.make_inputs(cfg)
    import torch
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, torch.from_numpy(d.orbitals).cuda(),
                   torch.from_numpy(d.ip_index).cuda())
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    x = ko.ip_values(d.orbitals, d.ip_index)
    w = np.stack([ctx.get_kernel(q) for q in range(cfg.n_k)])
    _check(cfg, ctx, x, w, [1, 2, 5, 7], ["fp64", "fp32", "bf16x3"])
    ctx.close()


@pytest.mark.parametrize("prec", ["bf16x3", "bf16"])
@pytest.mark.parametrize("n_ip", [33, 72, 129])
def test_small_bf16_tiles_same_bits(prec, n_ip):
    """Few 64 x 64 tiles take the small-tile kernel, many the 128 x 128 ones:
    a fragment alone and in a batch of over two rounds of tiles gets the same
    sums in the same order, so the same bits."""
    import torch
    cfg, ctx, x, w = _context(n_ip)
    sizes = [1, 5, 9, 12] + [40] * 4              # 4 x 325 tiles of 64 in the large ones alone
    dev = [torch.from_numpy(inp.make_fragment(cfg, f, n)).cuda() for f, n in enumerate(sizes)]
    batch = ctx.fragment_eri(dev, prec)
    for f in range(4):
        one = ctx.fragment_eri([dev[f]], prec)[0]
        assert torch.equal(one, batch[f]), (sizes[f], float((one - batch[f]).abs().max()))
    ctx.close()


@pytest.mark.parametrize("kmesh", [(6, 6, 6), (8, 8, 8)])
@pytest.mark.parametrize("n_ip", [7, 16, 19])
def test_jk_cubes(kmesh, n_ip):
    """J and K on the meshes whose exchange convolution keeps W's lines in
    registers, at element counts that do and do not fill its tiles; 1e-11
    relative given the GPU's W (FP64 k transforms of N_IP^2 elements)."""
    import paper_2601_16379_amd as pkg
    from oracle import hf
    cfg = dataclasses.replace(inp.get_config("t_small_k2"), kmesh=kmesh, n_ip=n_ip)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, d.orbitals, d.ip_index)
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    x = ko.ip_values(d.orbitals, d.ip_index)
    w = np.stack([ctx.get_kernel(q) for q in range(cfg.n_k)])
    dm = inp.make_density(cfg)
    j, k = ctx.hf_jk(dm)
    ks = [0, 1, cfg.n_k // 2 + 3, cfg.n_k - 1]
    k_ref, j_ref = hf.exchange_at(x, w, dm, cfg.kmesh, ks), hf.coulomb(x, w, dm)
    assert np.max(np.abs(k[ks] - k_ref)) <= 1e-11 * np.max(np.abs(k_ref))
    assert np.max(np.abs(j - j_ref)) <= 1e-11 * np.max(np.abs(j_ref))
    ctx.close()


@pytest.mark.parametrize("n", [6, 8, 10, 20, 24, 30, 36, 60])
def test_grid_transform_sizes(n):
    """Cubic grids of two small factors (in-place slab transform; ragged last
    blocks of slabs) and of none (60): Pi^q W^q Pi^q against the oracle's V^q
    within the bound of test_factor_edges, a q with phases included."""
    import paper_2601_16379_amd as pkg
    n_ip = 9
    cfg = dataclasses.replace(inp.get_config("t_small_k2"), grid=(n, n, n), kmesh=(2, 1, 1), n_ip=n_ip)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, d.orbitals, d.ip_index)
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    x = ko.ip_values(d.orbitals, d.ip_index)
    for q in (0, 1):
        pi, w = ctx.get_metric(q), ctx.get_kernel(q)
        v = ko.coulomb_kernel_of(ko.rhs(x, d.orbitals, cfg.kmesh, [q])[0], d.lattice, cfg.grid, cfg.kmesh, q)
        ev = np.linalg.eigvalsh(pi)
        bound = max(8 * n_ip * 2.0 ** -53 * ev[-1] / ev[0], 1e-12)
        err = np.max(np.abs(pi @ w @ pi - v)) / np.max(np.abs(v))
        assert ev[0] > 0 and err <= bound, (q, err, bound)
    ctx.close()


def test_idle_buffers_yield_to_fragment_workspace():
    """Buffers kept after a J/K build go back before the fragment workspace
    grows: the memory a fragment call leaves free does not depend on an earlier
    build."""
    import torch
    free = []
    for build in (False, True):
        cfg, ctx, x, w = _context(500)
        dev = [torch.from_numpy(inp.make_fragment(cfg, 0, 40)).cuda()]
        if build:
            ctx.hf_jk(inp.make_density(cfg))
        ctx.fragment_eri(dev, "fp64")
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free.append(torch.cuda.mem_get_info()[0])
        ctx.close()
    assert abs(free[0] - free[1]) <= 16 << 20, free      # rho alone is 8 x 500 x 500 x 16 bytes = 32 MB
