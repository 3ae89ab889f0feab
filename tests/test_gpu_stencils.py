"""Spread, gather and reciprocal force kernels at every chunk width (the split of a
wavefront's lanes over right-hand sides, stencil rows and atoms changes with it), every
spline order, ragged atom counts and grids that are no multiple of the 4-point tile, against
the oracle. Tolerances as in the parity tests: the reciprocal part alone 1e-11 in float64 and
1e-5 in mixed precision; forces 1e-7 and 1e-5 of the largest."""
import pytest
import torch

import synth
from oracle import lanczos as olz
from oracle import method as om

pytestmark = pytest.mark.gpu

A = synth.ANGSTROM_BOHR


def _plan(s, prec, block, p, grid, chunk=0, **kw):
    import paper_2307_02278_amd as P
    ds = P.DeviceSystem(s.pos, s.cell, s.alpha, s.omega, s.rvdw)
    if chunk:
        kw.update(tune=P.TUNE_GIVEN, shape=dict(overlap=1, grid_chunk=chunk))
    return P.Plan([ds], P.Params(ewald_tau=0.35 * synth.BOHR_ANGSTROM, real_cutoff=9.0 * A,
                                 grid=grid, spline_order=p, block=block, precision=prec, **kw))


def _op(s, plan, pos=None):
    inf = plan.info(0)
    mp = om.MethodParams(tau=inf.tau, r_pair=inf.r_pair, grid=tuple(inf.grid),
                         order=inf.spline_order, beta=0.83, d=6.0)
    return om.Operator(s, mp) if pos is None else om.Operator(s, mp, pos=pos)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("block,chunk,p", [(1, 0, 6), (1, 0, 4), (2, 0, 8), (4, 0, 6), (8, 0, 4),
                                           (8, 2, 6), (16, 0, 8), (32, 8, 6), (32, 32, 6),
                                           (64, 32, 4), (64, 64, 8)])
def test_reciprocal_part_at_every_chunk_width(block, chunk, p, prec):
    s = synth.triclinic_random(n=37, seed=5)
    plan = _plan(s, prec, block, p, (18, 20, 30), chunk, n_probes=block, n_steps=2)
    nr = min(block, 5)
    v = torch.randn(nr, s.n, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(2))
    got = plan.matvec(v.cuda(), components=4).cpu()
    plan.check()
    want = _op(s, plan)(v.permute(1, 2, 0), 4).permute(2, 0, 1)
    err = float(((got - want).abs().amax(dim=(1, 2)) / want.abs().amax(dim=(1, 2))).max())
    assert err < (1e-11 if prec == 0 else 1e-5), err


@pytest.mark.parametrize("prec,block,p", [(0, 4, 4), (0, 8, 8), (1, 4, 6), (1, 16, 8), (1, 32, 4)])
def test_forces_at_narrow_chunks(prec, block, p):
    s = synth.tiny_random(seed=4, n=11, L_ang=6.0, dmin_ang=1.8)
    m = 3
    plan = _plan(s, prec, block, p, (16, 18, 20), n_probes=block, n_steps=m, want_forces=True)
    e, f = plan.execute(forces=True)
    plan.check()
    pos = torch.tensor(s.pos, requires_grad=True)
    ref = olz.slq(_op(s, plan, pos), s.n, s.omega, seed=12345, n_probes=block, m=m,
                  reorth="none")
    (g,) = torch.autograd.grad(ref.energy, pos)
    ferr = float((f.cpu() + g).abs().max() / g.abs().max())
    assert ferr < (1e-7 if prec == 0 else 1e-5), ferr
