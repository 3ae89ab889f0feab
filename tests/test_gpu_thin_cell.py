"""A cell so thin that the cutoff spans more than 511 (and 1023) cells of it: the neighbour scan of the
narrow blocks and of the screening operator has no limit on the cell offsets."""
import numpy as np
import pytest
import torch

import synth
from oracle import method as om
from oracle import scs as osc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_narrow_block_and_screening_over_many_images(axis):
    import paper_2307_02278_amd as P
    edge = np.array([30.0, 30.0, 30.0])
    edge[axis] = 0.06
    s = synth.System("thin", np.array([[3.0, 4.0, 0.01], [10.0, 0.02, 21.0]]), np.diag(edge),
                     np.array([1e-7, 2e-7]), np.array([0.5, 0.6]), np.array([3.0, 3.3]))
    grid = [12, 12, 12]
    plan = P.Plan([P.DeviceSystem(s.pos, s.cell, s.alpha, s.omega, s.rvdw)],
                  P.Params(ewald_tau=0.1, real_cutoff=75.0, grid=tuple(grid), spline_order=4,
                           n_probes=1, n_steps=2, block=1, precision=P.PREC_FP64,
                           damp_tol=-1.0))
    inf = plan.info(0)
    op = om.Operator(s, om.MethodParams(tau=inf.tau, r_pair=inf.r_pair, grid=tuple(inf.grid),
                                        order=inf.spline_order))
    v = torch.randn(1, 2, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(1))
    got = plan.matvec(v.cuda(), components=2).cpu()
    want = op(v.permute(1, 2, 0), 2).permute(2, 0, 1)
    err = float((got - want).abs().max() / want.abs().max())
    assert err < 1e-11, err
    # polarizabilities small enough that the screening matrix is positive definite
    a, o, r, _ = plan.scs(n_freq=3, tol=1e-13)
    ra, ro, rr, _, _ = osc.scs(s, 0.83, 6.0, inf.r_pair, n_freq=3)
    for x, y in ((a, ra), (o, ro), (r, rr)):
        assert float(((x.cpu() - y).abs() / y.abs()).max()) < 1e-10
