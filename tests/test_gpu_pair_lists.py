"""The direct-space sum over its lists, against the oracle's direct field: the neighbour
list of the narrow blocks at the edges of its wavefront split, with a list that later
positions outgrow (the targets past its capacity are then summed on the fly), and with no
pair in range at all. Tolerances as in the parity tests: 1e-11 in float64 (differently
ordered sums), 1e-5 for the direct part alone in mixed precision."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import synth
from oracle import method as om

pytestmark = pytest.mark.gpu

A = synth.ANGSTROM_BOHR
TOL = {0: 1e-11, 1: 1e-5}


def _random(n, L_ang, seed):
    rng = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1 / 3)))
    at = rng.choice(m ** 3, n, replace=False)
    f = np.stack([at % m, (at // m) % m, at // (m * m)], 1) + rng.uniform(0.2, 0.8, (n, 3))
    return synth.System("random", f / m * L_ang * A, np.eye(3) * L_ang * A,
                        rng.uniform(5, 15, n), rng.uniform(0.3, 0.7, n), rng.uniform(3, 4, n))


def _cutoff(s, rc_ang):
    """A cutoff (bohr) near rc_ang with no pair within 1e-6 of it, relative (a float32
    distance is good to about 3e-7): a pair at the
    cutoff itself belongs to the float32 sum or not by its rounded distance, while the bare
    cutoff of these plans (no damping tail) leaves it a finite tensor."""
    L = s.cell[0, 0]
    tree = cKDTree(s.pos % L, boxsize=L)
    p = tree.query_pairs(min(rc_ang * A * 1.001, 0.499 * L), output_type="ndarray")
    d = s.pos[p[:, 0]] - s.pos[p[:, 1]]
    d -= L * np.round(d / L)
    r = np.sort(np.concatenate([np.linalg.norm(d, axis=1), np.array([0.999, 1.001]) * rc_ang * A]))
    r = r[r >= 0.999 * rc_ang * A]
    k = int(np.argmax(np.diff(r)))
    assert r[k + 1] - r[k] > 2e-6 * r[k]
    return 0.5 * (r[k] + r[k + 1])


def _plan(s, prec, block, rc_ang, grid):
    import paper_2307_02278_amd as P
    ds = P.DeviceSystem(s.pos, s.cell, s.alpha, s.omega, s.rvdw)
    return P.Plan([ds], P.Params(real_cutoff=_cutoff(s, rc_ang), grid=grid, n_probes=block, n_steps=2,
                                 block=block, precision=prec, damp_tol=-1.0))


def _direct_error(plan, s, block):
    inf = plan.info(0)
    op = om.Operator(s, om.MethodParams(tau=inf.tau, r_pair=inf.r_pair, grid=tuple(inf.grid),
                                        order=inf.spline_order, beta=0.83, d=6.0))
    nr = min(block, 4)
    v = torch.randn(nr, s.n, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(3))
    got = plan.matvec(v.cuda(), components=2).cpu()
    want = op(v.permute(1, 2, 0), 2).permute(2, 0, 1)
    plan.check()
    den = want.abs().amax(dim=(1, 2))
    assert float(den.min()) > 0.0
    return float(((got - want).abs().amax(dim=(1, 2)) / den).max())


# 8191 and 8192 atoms: four wavefronts per target, then one; 8195: a ragged last work-group
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,block", [(5, 1), (63, 2), (515, 4), (515, 8), (8191, 1), (8192, 2),
                                     (8195, 8)])
def test_neighbour_list_matches_the_oracle(n, block, prec):
    s = _random(n, (n / 0.05) ** (1 / 3), seed=n)
    plan = _plan(s, prec, block, 6.0, (24, 24, 24))
    assert _direct_error(plan, s, block) < TOL[prec]


@pytest.mark.parametrize("prec,block", [(0, 1), (0, 8), (1, 2)])
def test_positions_denser_than_the_neighbour_list(prec, block):
    """Half of the atoms moved into a corner: their targets have more pairs than the list
    holds, the others fewer; every pair still counts, and the next positions use the list."""
    s0 = _random(400, 40.0, seed=8)
    plan = _plan(s0, prec, block, 6.0, (24, 24, 24))
    pos1 = s0.pos.copy()
    pos1[::2] = _random(200, 15.0, seed=9).pos
    plan.set_positions(torch.as_tensor(pos1).cuda())
    s1 = synth.System("corner", pos1, s0.cell, s0.alpha, s0.omega, s0.rvdw)
    assert _direct_error(plan, s1, block) < TOL[prec]
    plan.set_positions(torch.as_tensor(s0.pos).cuda())
    assert _direct_error(plan, s0, block) < TOL[prec]


def test_no_pair_in_range():
    s = synth.one_atom(at=(1.0, 2.0, 3.0), L_ang=12.0)
    plan = _plan(s, 0, 1, 5.0, (16, 16, 16))
    v = torch.ones(1, 1, 3, dtype=torch.float64).cuda()
    assert float(plan.matvec(v, components=2).abs().max()) == 0.0


# one group (its list in 16 parts, some of them empty), a ragged second group, 16 groups and
# enough groups for one part; every width of the float64 and the narrow mixed wavefronts
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,block", [(5, 16), (17, 32), (250, 16), (250, 64), (250, 128),
                                     (131, 256), (8200, 16), (16400, 32)])
def test_tensor_list_parts_match_the_oracle(n, block, prec):
    s = _random(n, (n / 0.05) ** (1 / 3), seed=n + 1)
    plan = _plan(s, prec, block, 6.0, (24, 24, 24))
    assert _direct_error(plan, s, block) < TOL[prec]
