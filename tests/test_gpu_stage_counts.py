"""Stage counters count launches: one per transform pass, and only the three that exist
where the transforms run by planes (small float grids with K2 = K3)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,grid,planes", [(1, (24, 24, 24), True), (1, (24, 20, 24), False),
                                              (0, (24, 24, 24), False)])
def test_transform_passes_are_counted_as_launched(prec, grid, planes):
    import paper_2307_02278_amd as P
    rng = np.random.default_rng(1)
    n = 50
    ds = [P.DeviceSystem(rng.uniform(0, 25, (n, 3)), np.eye(3) * 25.0, np.full(n, 6.0),
                         np.full(n, 0.5), np.full(n, 3.2))]
    plan = P.Plan(ds, P.Params(real_cutoff=10.0, grid=grid, n_probes=16, n_steps=3, block=16,
                               precision=prec, want_forces=True))
    plan.set_timing(True)
    plan.matvec(torch.randn(16, n, 3, dtype=torch.float64).cuda())
    got = {k: c for k, (_, c) in plan.stage_times().items()}
    want = {"fft_x": 1, "fft_y": 0 if planes else 1, "fft_z_conv": 1,
            "ifft_y": 0 if planes else 1, "ifft_x": 1, "pair": 1, "spread": 1, "gather": 1}
    assert {k: got[k] for k in want} == want
    plan.execute(forces=True)
    got = {k: c for k, (_, c) in plan.stage_times().items()}
    # forward: 3 matvecs; reverse: the grids of p and of q at each of 3 steps, the pair sum
    # of p at the two steps whose adjoint matvec is read
    passes = 3 + 2 * 3
    want = {"fft_x": passes, "fft_y": 0 if planes else passes, "fft_z_conv": passes,
            "ifft_y": 0 if planes else passes, "ifft_x": passes, "pair": 5, "gather": 3}
    assert {k: got[k] for k in want} == want
