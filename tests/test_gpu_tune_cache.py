"""The file of measured shapes: a shape is taken from it only for the kernels and the direct
cutoff that it was measured with. Lines of other builds (no kernel generation, or another
one) are read without an error and measured anew."""
import json

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _plan(cache, rc=11.0):
    import paper_2307_02278_amd as P
    rng = np.random.default_rng(2)
    n = 300
    ds = [P.DeviceSystem(rng.uniform(0, 30, (n, 3)), np.eye(3) * 30.0, np.full(n, 6.0),
                         np.full(n, 0.5), np.full(n, 3.2))]
    return P.Plan(ds, P.Params(real_cutoff=rc, grid=(24, 24, 24), n_probes=64, n_steps=3,
                               block=64, precision=P.PREC_MIXED, tune=P.TUNE_MEASURE,
                               tune_cache=cache, damp_tol=-1.0))


def test_shapes_of_other_kernels_and_cutoffs_are_measured_anew(tmp_path):
    cache = str(tmp_path / "shapes.jsonl")
    plan = _plan(cache)
    assert plan.info(0).shape_source == 1
    line = json.loads(open(cache).read())
    assert _plan(cache).info(0).shape_source == 2
    # the same key as an earlier build wrote it, and with another kernel generation
    old = {k: line[k] for k in ("key", "pair_wg_per_cu", "pair_subsets", "grid_chunk", "overlap",
                                "gather_waves", "spread_mode", "pair_mode", "matvec_ms")}
    for extra in ({}, {k: line[k] + 1 for k in line if k == "kernels"}):
        with open(cache, "w") as f:
            f.write(json.dumps({**line, **old, **extra} if extra else old) + "\n")
        assert _plan(cache).info(0).shape_source == 1
        assert _plan(cache).info(0).shape_source == 2
    assert _plan(cache, rc=9.0).info(0).shape_source == 1
    assert _plan(cache, rc=9.0).info(0).shape_source == 2
    assert _plan(cache).info(0).shape_source == 2
