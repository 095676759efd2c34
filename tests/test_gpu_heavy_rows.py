"""Rows and segments whose Gram is dealt to several wavefronts: degrees on both
sides of the limit (256 ratings on a matrix this small), with a last wavefront
that is left a few ratings or none, against the oracle at the bars of the other
single steps."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


DEGREES = [3, 255, 256, 257, 258, 320, 384, 385, 513, 608, 640, 641, 1024, 1025, 1026, 2051, 2900, 0, 1]


def _columns(degrees, M, seed):
    """A matrix whose movies have the given degrees (users at random)."""
    rng = np.random.default_rng(seed)
    rows = np.concatenate([np.sort(rng.choice(M, d, replace=False)) for d in degrees])
    cols = np.repeat(np.arange(len(degrees)), degrees)
    vals = rng.standard_normal(len(rows)) + 3.0
    return synth._assemble("heavy-columns", M, len(degrees), rows.astype(np.int64), cols, vals.astype(np.float32),
                           0.0, rng, 8)


@pytest.mark.parametrize("prec,K", [("fp32", 9), ("fp32", 16), ("fp32", 32), ("fp32", 36), ("fp32", 64), ("fp32", 100), ("fp32", 128), ("bf16", 20),
                                    ("bf16", 96), ("bf16", 100)])
@pytest.mark.parametrize("split", [0, 1025])
def test_heavy_rows(bp, orc, prec, K, split):  # noqa: F811
    r = _columns(DEGREES, 3000, K)
    err, _, _ = single_step(bp, orc, r, K, prec, bp.SIDE_V, split=split)
    assert err.max() <= TOL[prec]


@pytest.mark.parametrize("K", [33, 48, 64])
def test_heavy_rows_column_kernel(bp, orc, K):  # noqa: F811
    """The column-per-lane kernel above K = 32, where a plan asks for it."""
    r = _columns(DEGREES, 3000, K)
    err, _, _ = single_step(bp, orc, r, K, "fp32", bp.SIDE_V, plan=(1025, 64, 0))
    assert err.max() <= TOL["fp32"]
