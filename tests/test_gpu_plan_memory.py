"""The neighbour lists of narrow blocks are optional (the kernel can sum over the cells), so
they never take the memory of what a plan cannot do without: a batch whose buffers fit is
accepted although its lists no longer do, and gives the same direct sum."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

pytestmark = pytest.mark.gpu

RC, BLOCK, STEPS = 22.0, 8, 120


def _box(seed):
    rng = np.random.default_rng(seed)
    m, side = 28, 112.0
    at = np.arange(m ** 3)
    f = np.stack([at % m, (at // m) % m, at // (m * m)], 1) + rng.uniform(0.4, 0.6, (m ** 3, 3))
    n = m ** 3
    return (f / m * side, np.eye(3) * side, np.full(n, 6.0), np.full(n, 0.5), np.full(n, 3.2))


def _plan(boxes):
    import paper_2307_02278_amd as P
    return P.Plan([P.DeviceSystem(*b) for b in boxes],
                  P.Params(real_cutoff=RC, grid=(48, 48, 48), n_probes=BLOCK, n_steps=STEPS,
                           block=BLOCK, precision=P.PREC_FP64, damp_tol=-1.0))


def test_lists_leave_room_for_the_other_systems():
    boxes = [_box(1), _box(2)]
    n = len(boxes[0][0])
    v = torch.randn(BLOCK, n, 3, dtype=torch.float64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(4))
    free = _plan(boxes)
    want = [free.matvec(v, sys=k, components=2).cpu() for k in range(2)]
    total = sum(free.info(k).workspace_bytes for k in range(2))
    free.close()
    lists = 0
    for b in boxes:
        t = cKDTree(b[0] % b[1][0, 0], boxsize=b[1][0, 0])
        most = max(len(x) for x in t.query_ball_point(b[0] % b[1][0, 0], RC, workers=8)) - 1
        lists += n * (most + most // 4 + 16) * 24
    # memory for everything but the lists, and a third of those
    torch.cuda.empty_cache()
    leave = total - lists + lists // 3
    filler = []
    for _ in range(4):  # (the runtime hands memory it kept back as it sees need)
        rest = torch.cuda.mem_get_info()[0] - leave
        if rest > (64 << 20):
            filler.append(torch.empty(rest, dtype=torch.uint8, device="cuda"))
    try:
        plan = _plan(boxes)
        got = [plan.matvec(v, sys=k, components=2).cpu() for k in range(2)]
        plan.check()
        plan.close()
    finally:
        filler.clear()
        torch.cuda.empty_cache()
    for a, b in zip(got, want):
        assert float((a - b).abs().max() / b.abs().max()) < 1e-11
