"""Transforms by y-z planes (small float grids with K2 = K3): the reciprocal part of C against
a float64 plan of the same grid, whose transforms run pass by pass. Sizes: one to eight planes
per work-group, line counts that are not a multiple of 8, odd half lengths, every chunk width,
and one grid just above the size rule. The float transforms of 3 log2 K stages each way lose
about (6 log2 K) 2^-24 = 2e-6 of the largest value at most, typically a tenth of it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,block", [
    ((16, 16, 16), 16), ((24, 18, 18), 64), ((20, 30, 30), 32), ((32, 36, 36), 64),
    ((50, 50, 50), 16), ((36, 54, 54), 16), ((64, 72, 72), 16), ((40, 40, 40), 128),
    ((48, 48, 48), 64), ((24, 20, 24), 64)])
def test_planes_match_float64(grid, block):
    import paper_2307_02278_amd as P
    rng = np.random.default_rng(sum(grid) + block)
    n, side = 150, 28.0
    ds = [P.DeviceSystem(rng.uniform(0, side, (n, 3)), np.eye(3) * side, rng.uniform(4, 9, n),
                         rng.uniform(.3, .7, n), rng.uniform(3.0, 3.6, n))]
    v = torch.randn(block, n, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(2))
    out = []
    for prec in (P.PREC_MIXED, P.PREC_FP64):
        plan = P.Plan(ds, P.Params(real_cutoff=13.0, grid=grid, n_probes=block, n_steps=4,
                                   block=block, precision=prec))
        for _ in range(2):
            r = plan.matvec(v.cuda(), components=P.C_REC)
        out.append(r.cpu())
        plan.close()
    err = float((out[0] - out[1]).abs().max() / out[1].abs().max())
    print(grid, block, f"{err:.2e}")
    assert err < 2e-6
