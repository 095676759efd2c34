"""The packed FP64 kernel (K <= 16, more than 10,240 light rows) with items that
four wavefronts share: whole rows and segments of split rows just above the
limit of 256 ratings and far above it.  Single steps against the oracle at the
FP64 bar."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu

HEAVY = [257, 258, 513, 1025, 2900, 256, 255, 300, 301]


def _users(M, N, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 6, M)
    deg[: len(HEAVY)] = HEAVY
    rows = np.repeat(np.arange(M), deg)
    cols = np.concatenate([np.sort(rng.choice(N, d, replace=False)) for d in deg])
    vals = (rng.standard_normal(len(rows)) + 3.0).astype(np.float32)
    return synth._assemble("heavy-users", M, N, rows.astype(np.int64), cols.astype(np.int64), vals, 0.0, rng, 8)


@pytest.mark.parametrize("K", [1, 7, 15, 16])
@pytest.mark.parametrize("split", [0, 300, 600])
def test_packed_heavy_items(bp, orc, K, split):  # noqa: F811
    r = _users(10403, 3000, K)
    s = bp.Sampler(r, K, prec="fp64", seed=1, split_threshold=split)
    assert s.get_plan(bp.SIDE_U)[1] == (sum(d > split for d in HEAVY) if split else 1)
    s.close()
    err, _, _ = single_step(bp, orc, r, K, "fp64", bp.SIDE_U, split=split)
    assert err.max() <= TOL["fp64"]
