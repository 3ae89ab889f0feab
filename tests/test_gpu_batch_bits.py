"""A system's results do not depend on the systems that share its plan: energy, forces and
C v of a box come out the same bits alone and beside others (a batch runs without the side
stream, which changes no bit). 2187 atoms are 137 target groups, enough that the direct sum
is split into fewer parts than its limit in either precision."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _box(n, side, seed):
    rng = np.random.default_rng(seed)
    m = int(np.ceil(n ** (1 / 3)))
    at = rng.choice(m ** 3, n, replace=False)
    f = np.stack([at % m, (at // m) % m, at // (m * m)], 1) + rng.uniform(0.3, 0.7, (n, 3))
    return (f / m * side, np.eye(3) * side, rng.uniform(4, 8, n), rng.uniform(0.4, 0.6, n),
            rng.uniform(3.0, 3.6, n))


@pytest.mark.parametrize("prec,block", [(0, 16), (1, 16), (1, 64)])
def test_same_bits_alone_and_in_a_batch(prec, block):
    import paper_2307_02278_amd as P
    boxes = [P.DeviceSystem(*_box(2187, 62.0, 1)), P.DeviceSystem(*_box(64, 19.0, 2)),
             P.DeviceSystem(*_box(512, 38.0, 3)), P.DeviceSystem(*_box(100, 23.0, 4))]
    v = torch.randn(block, 2187, 3, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(5))
    out = []
    for systems in (boxes[:1], boxes[:2], boxes):
        plan = P.Plan(systems, P.Params(real_cutoff=13.0, grid=(36, 36, 36), n_probes=block,
                                        n_steps=4, block=block, precision=prec,
                                        want_forces=True))
        e, f = plan.execute(forces=True)
        plan.check()
        out.append((e[:1].cpu(), f[:2187].cpu(), plan.matvec(v, sys=0).cpu()))
        plan.close()
    for got in out[1:]:
        for a, b in zip(out[0], got):
            assert torch.equal(a, b)
