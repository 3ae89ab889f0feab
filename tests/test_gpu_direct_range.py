"""The direct field of dipoles outside the range of ordinary ones. A pair out of range adds
nothing to it, also when the source's dipole is infinite or not a number: the targets out of
its range and the other right-hand sides keep their values. Dipoles at the ends of float's
range (above the largest bfloat16, and so small that their last bits are below the smallest)
give the field that float products give: 1e-5 of its largest element, the bound of the
direct part in mixed precision (1e-11 in float64)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = {0: 1e-11, 1: 1e-5}
N, RC = 600, 11.0


def _box(seed=3):
    rng = np.random.default_rng(seed)
    side, m = 43.0, 9
    at = rng.choice(m ** 3, N, replace=False)
    f = np.stack([at % m, (at // m) % m, at // (m * m)], 1) + rng.uniform(0.25, 0.75, (N, 3))
    return (f / m * side, np.eye(3) * side, rng.uniform(5, 15, N), rng.uniform(0.3, 0.7, N),
            rng.uniform(3, 4, N))


def _plan(prec, block):
    import paper_2307_02278_amd as P
    return P.Plan([P.DeviceSystem(*_box())],
                  P.Params(real_cutoff=RC, grid=(24, 24, 24), n_probes=block, n_steps=2,
                           block=block, precision=prec, damp_tol=-1.0))


def _distances(j):
    pos, cell = _box()[:2]
    d = pos - pos[j]
    d -= cell[0, 0] * np.round(d / cell[0, 0])
    return np.linalg.norm(d, axis=1)


WIDTHS = [(0, 8), (0, 16), (0, 32), (0, 64), (0, 128), (0, 256), (1, 8), (1, 16), (1, 32),
          (1, 64), (1, 128), (1, 256)]


@pytest.mark.parametrize("prec,block", WIDTHS)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_non_finite_dipole_reaches_its_own_pairs_only(prec, block, value):
    plan = _plan(prec, block)
    g = torch.Generator().manual_seed(block)
    v = torch.randn(block, N, 3, dtype=torch.float64, generator=g)
    col, atom = block - 2, 77
    v[col, atom] = 0.0
    want = plan.matvec(v.cuda(), components=2).cpu()
    v[col, atom, 1] = value
    got = plan.matvec(v.cuda(), components=2).cpu()
    r = _distances(atom)
    far = torch.tensor((r > RC * (1 + 1e-5)) | (r == 0.0))
    near = torch.tensor((r < RC * (1 - 1e-5)) & (r > 0.0))
    assert int(near.sum()) > 10 and int(far.sum()) > 300
    assert not torch.isfinite(got[col][near]).any(dim=1).all()
    assert not torch.isfinite(got[col][near]).all(dim=1).any()
    assert torch.isfinite(got[col][far]).all()
    err = float((got[col][far] - want[col][far]).abs().max() / want[col].abs().max())
    assert err < TOL[prec], err
    others = [c for c in range(block) if c != col]
    assert torch.equal(got[others], want[others])


@pytest.mark.parametrize("block,size", [(b, x) for b in (16, 32, 64, 128, 256)
                                        for x in (3.397e38, 1e-34, 1e-36, 1e-37)]
                         + [(8, 1e-34), (8, 1e-36)])
def test_dipoles_at_the_ends_of_the_float_range(block, size):
    """One column has dipoles of that size (a single one for the largest, so that the sums
    stay finite), the others ordinary ones."""
    box = _box()
    gi = box[3] * np.sqrt(box[2])
    g = torch.Generator().manual_seed(block)
    v = torch.randn(block, N, 3, dtype=torch.float64, generator=g)
    col = block - 1
    if size > 1.0:
        v[col] = 0.0
        v[col, 123, 2] = size / gi[123]
    else:
        v[col] *= torch.tensor(size / gi)[:, None]
    got = _plan(1, block).matvec(v.cuda(), components=2).cpu()
    want = _plan(0, 8).matvec(v[col:].cuda(), components=2).cpu()[0]
    assert torch.isfinite(got).all()
    err = float((got[col] - want).abs().max() / want.abs().max())
    print(f"block {block} size {size}: {err:.2e}")
    assert err < 1e-5
