"""The rank-one path on fewer rows than a group of 16, a wavefront's four, or one:
every user has few ratings, so all of them take it (asserted), a single step
against the oracle at the FP32 bar."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,low", [(7, 4), (17, 16), (32, 8), (48, 8), (64, 16)])
@pytest.mark.parametrize("degrees", [[3], [0], [4, 0, 3], [1, 4, 2, 4, 0], [4] * 17])
def test_lowrank_tiny(bp, orc, K, low, degrees):  # noqa: F811
    rng = np.random.default_rng(K)
    deg = np.array(degrees) * (low // 4)
    rows = np.repeat(np.arange(len(deg)), deg)
    cols = np.concatenate([rng.choice(40, d, replace=False) for d in deg])
    vals = (rng.standard_normal(len(rows)) + 3.0).astype(np.float32)
    r = synth._assemble("tiny", len(deg), 40, rows.astype(np.int64), cols.astype(np.int64), vals, 0.0, rng, 8)
    plan = (2048, 32, low)
    s = bp.Sampler(r, K, prec="fp32", seed=1)
    s.set_plan(*plan)
    assert s.lowrank_rows(bp.SIDE_U) == len(deg)
    s.close()
    err, _, _ = single_step(bp, orc, r, K, "fp32", bp.SIDE_U, plan=plan)
    assert err.max() <= TOL["fp32"]
