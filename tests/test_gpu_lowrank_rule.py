"""Which sides take the rank-one path above K = 64 by default, and its launches at
their edges: rows of at most 4 ratings in the launch of the others (up to 4096)
or in their own, one and two rounds of the transform.  Single steps against the
oracle at the FP32 bar."""
import numpy as np
import pytest

from test_gpu_lowrank_wide import _sparse
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,M,N,taken", [
    (65, 6001, 12, True), (81, 9001, 700, True), (128, 12001, 2500, True), (65, 30011, 4001, True),
    (65, 97, 12, False), (128, 97, 12, False), (65, 3001, 150, False), (112, 2001, 150, False),
    (128, 2901, 150, True), (65, 12001, 12000, False),
])
def test_lowrank_rule(bp, orc, K, M, N, taken):  # noqa: F811
    r = _sparse(M, N, K)
    deg = np.diff(r.csr_ptr)
    s = bp.Sampler(r, K, prec="fp32", seed=3)
    assert s.lowrank_rows(bp.SIDE_U) == ((deg <= 8).sum() if taken else 0)
    s.close()
    rows = np.unique(np.concatenate([np.arange(0, M, max(1, M // 800)), [M - 1]]))
    err, _, _ = single_step(bp, orc, r, K, "fp32", bp.SIDE_U, rows=rows)
    assert err.max() <= TOL["fp32"]
