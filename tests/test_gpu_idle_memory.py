"""Device memory that contexts keep between J/K, MP2 and dRPA calls."""
import dataclasses

import numpy as np
import pytest

import isdf_inputs as inp

pytestmark = pytest.mark.gpu

N_IP = 500
RHO = 8 * N_IP * N_IP * 16       # bytes of one matrix a k point (2x2x2 mesh): 32 MB


def _context():
    import torch
    import paper_2601_16379_amd as pkg
    cfg = dataclasses.replace(inp.get_config("t_small_k2"), n_ip=N_IP)
    d = inp.make_inputs(cfg)
    ctx = pkg.Isdf(d.lattice, cfg.grid, cfg.kmesh, torch.from_numpy(d.orbitals).cuda(),
                   torch.from_numpy(d.ip_index).cuda())
    ctx.fit()
    ctx.coulomb_kernel("fp64")
    return cfg, ctx


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_idle_buffers_yield_to_another_context():
    """A fragment workspace is planned as if the idle buffers of every context
    were free, so they go back before it grows: what a fragment call leaves free
    does not depend on an earlier build of another context."""
    import torch
    free = []
    for build in (False, True):
        cfg, one = _context()
        _, two = _context()
        if build:
            one.hf_jk(inp.make_density(cfg))
        two.fragment_eri([torch.from_numpy(inp.make_fragment(cfg, 0, 40)).cuda()], "fp64")
        free.append(_free())
        one.close()
        two.close()
    assert abs(free[0] - free[1]) <= RHO // 2, free


def test_failed_call_keeps_nothing():
    """A call that fails after its workspace was allocated (a transform whose
    polarisabilities overflow) leaves the device memory as it found it."""
    import paper_2601_16379_amd as pkg
    cfg, ctx = _context()
    c, e, n_occ = inp.make_mo(cfg)
    tau, _ = inp.laplace_grid(3, 1.0)
    _, ow = inp.laplace_grid(2, 1.0)
    before = _free()
    with pytest.raises(pkg.IsdfError) as ex:
        ctx.drpa(c, e, n_occ, tau, ow, np.full((2, 3), 1e300 + 0j))
    assert ex.value.status == -4
    assert before - _free() <= RHO // 2
    ctx.close()


def _calls(cfg, ctx):
    """J/K, MP2 and dRPA with workspaces of several sizes, as functions."""
    c, e, n_occ = inp.make_mo(cfg)
    tau, tw = inp.laplace_grid(3, 1.0)
    om, ow = inp.laplace_grid(2, 1.0)
    g = inp.quadrature_transform(tau, tw, om)
    dm = inp.make_density(cfg)
    return {"jk": lambda: ctx.hf_jk(dm),
            "j": lambda: ctx.hf_jk(dm, want_k=False)[0],
            "mp2": lambda: ctx.sos_mp2(c, e, n_occ, tau, tw)["integrand"],
            "mp2 fewer": lambda: ctx.sos_mp2(np.ascontiguousarray(c[:, :, 1:5]), e[:, 1:5], 2, tau, tw)["integrand"],
            "drpa": lambda: ctx.drpa(c, e, n_occ, tau, ow, g)["integrand"],
            "drpa one": lambda: ctx.drpa(c, e, n_occ, tau, ow[:1], g[:1])["integrand"]}


def test_release_idle_hands_everything_back():
    cfg, ctx = _context()
    calls = _calls(cfg, ctx)
    for f in calls.values():              # the arenas and code of every call
        f()
    ctx.release_idle()
    before = _free()
    for name, f in calls.items():
        f()
        kept = before - _free()
        assert kept > RHO // 2 or name == "j", (name, kept)
        ctx.release_idle()
        assert before - _free() <= 4 << 20, name
    ctx.close()


def test_calls_in_turn_equal_calls_alone():
    """Results do not depend on what an earlier call of another size left in the
    buffers it handed on."""
    cfg, ctx = _context()
    calls = _calls(cfg, ctx)
    alone = {}
    for name, f in calls.items():
        ctx.release_idle()
        alone[name] = f()
    rng = np.random.default_rng(5)
    for name in rng.choice(list(calls), 30):
        for a, b in zip(np.atleast_1d(calls[name]()), np.atleast_1d(alone[name])):
            assert np.array_equal(a, b), name
    ctx.close()
