"""The tensor-list kernels where small tests do not reach: every right-hand side of wide
blocks, candidate ranges longer than one LDS chunk (1024), and launches with fewer
work-groups than target groups, so that each walks several. Against the oracle; tolerances
as in the parity tests, 1e-11 in float64 and 1e-5 for one part of C alone in mixed
precision."""
import numpy as np
import pytest
import torch

import synth
from oracle import method as om

pytestmark = pytest.mark.gpu

A = synth.ANGSTROM_BOHR
TOL = {0: 1e-11, 1: 1e-5}


def _random(n, seed):
    rng = np.random.default_rng(seed)
    side = (n / 0.05) ** (1 / 3)
    m = int(np.ceil(n ** (1 / 3)))
    at = rng.choice(m ** 3, n, replace=False)
    f = np.stack([at % m, (at // m) % m, at // (m * m)], 1) + rng.uniform(0.25, 0.75, (n, 3))
    return synth.System("random", f / m * side * A, np.eye(3) * side * A,
                        rng.uniform(5, 15, n), rng.uniform(0.3, 0.7, n), rng.uniform(3, 4, n))


def _plan(s, prec, block, rc_ang, grid=(24, 24, 24), shape=None, **kw):
    import paper_2307_02278_amd as P
    if shape is not None:
        kw.update(tune=P.TUNE_GIVEN, shape=shape)
    return P.Plan([P.DeviceSystem(s.pos, s.cell, s.alpha, s.omega, s.rvdw)],
                  P.Params(real_cutoff=rc_ang * A, grid=grid, n_probes=block, n_steps=2,
                           block=block, precision=prec, **kw))


def _error(plan, s, block, comp, columns):
    """All right-hand sides are filled; the given ones are compared."""
    inf = plan.info(0)
    op = om.Operator(s, om.MethodParams(tau=inf.tau, r_pair=inf.r_pair, grid=tuple(inf.grid),
                                        order=inf.spline_order, beta=0.83, d=6.0))
    v = torch.randn(block, s.n, 3, dtype=torch.float64,
                    generator=torch.Generator().manual_seed(block + s.n))
    got = plan.matvec(v.cuda(), components=comp).cpu()[columns]
    plan.check()
    want = op(v[columns].permute(1, 2, 0), comp).permute(2, 0, 1)
    return got, float(((got - want).abs().amax(dim=(1, 2)) / want.abs().amax(dim=(1, 2))).max())


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,block", [(17, 16), (40, 32), (250, 64), (131, 128), (40, 256)])
def test_every_right_hand_side_of_the_direct_sum(n, block, prec):
    s = _random(n, n)
    _, err = _error(_plan(s, prec, block, 6.0), s, block, 2, list(range(block)))
    assert err < TOL[prec], err


@pytest.mark.parametrize("prec,block,chunk", [(0, 32, 8), (0, 64, 16), (0, 256, 0), (1, 32, 8),
                                              (1, 64, 16), (1, 64, 2), (1, 256, 64)])
def test_every_right_hand_side_of_the_grid_chunks(prec, block, chunk):
    s = _random(37, 5)
    plan = _plan(s, prec, block, 5.0, (18, 20, 30), dict(grid_chunk=chunk))
    _, err = _error(plan, s, block, 4, list(range(block)))
    assert err < TOL[prec], err


# one part (more than 512 or 1024 groups), about 1400 candidates a group
@pytest.mark.parametrize("prec,n,block", [(1, 8300, 16), (1, 8300, 64), (1, 8300, 128),
                                          (0, 16500, 16)])
def test_candidate_lists_longer_than_one_chunk(prec, n, block):
    s = _random(n, 7)
    plan = _plan(s, prec, block, 16.0, damp_tol=-1.0)
    _, err = _error(plan, s, block, 2, [0, block // 2 + 1, block - 1])
    assert err < TOL[prec], err


# 188 groups in several parts and 521 groups in one, on 256 work-groups at most
@pytest.mark.parametrize("prec,n,block,mode", [(0, 3000, 16, 0), (1, 3000, 32, 0),
                                               (1, 3000, 64, 1), (1, 3000, 256, 1),
                                               (1, 3000, 128, 2), (1, 8330, 64, 1),
                                               (1, 8330, 16, 0), (0, 8330, 64, 0)])
def test_a_work_group_walks_several_groups(prec, n, block, mode):
    s = _random(n, 9)
    got = []
    for cap in (0, 1):
        plan = _plan(s, prec, block, 6.0, shape=dict(pair_wg_per_cu=cap, pair_mode=mode))
        r, err = _error(plan, s, block, 2, [0, block - 1])
        assert err < TOL[prec], err
        got.append(r)
    assert torch.equal(got[0], got[1])
