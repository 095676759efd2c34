"""The rank-one path above K = 64 (every component count per lane) and in groups
of 16 rows (fewer rows than a group, a ragged last group, several groups a
workgroup): single steps against the oracle at the FP32 bar (1e-4 a row), with
the prior set by the host and by the hyper draw."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


def _sparse(M, N, seed):
    """Users with 0 to 8 ratings, a few with more."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 9, M)
    deg[:: max(1, M // 5)] = 11
    rows = np.repeat(np.arange(M), deg)
    cols = np.concatenate([rng.choice(N, d, replace=False) for d in deg])
    vals = (rng.standard_normal(len(rows)) + 3.0).astype(np.float32)
    return synth._assemble("few-ratings", M, N, rows.astype(np.int64), cols.astype(np.int64), vals, 0.0, rng, 8)


@pytest.mark.parametrize("K", [65, 80, 81, 96, 100, 112, 113, 128])
@pytest.mark.parametrize("M", [97, 5003])
def test_lowrank_above_64(bp, orc, K, M):  # noqa: F811
    r = _sparse(M, 12, K)
    s = bp.Sampler(r, K, prec="fp32", seed=3)
    deg = np.diff(r.csr_ptr)
    paid = (deg <= 8).sum() * K / 3.0 > 4.0 * r.N
    assert s.lowrank_rows(bp.SIDE_U) == ((deg <= 8).sum() if paid else 0) and paid
    s.close()
    err, _, _ = single_step(bp, orc, r, K, "fp32", bp.SIDE_U)
    assert err.max() <= TOL["fp32"]


@pytest.mark.parametrize("K,low", [(7, 4), (17, 16), (48, 8), (64, 16)])
@pytest.mark.parametrize("M", [3, 33, 40003])
def test_lowrank_groups(bp, orc, K, low, M):  # noqa: F811
    r = _sparse(M, 40, K)
    err, _, _ = single_step(bp, orc, r, K, "fp32", bp.SIDE_U, plan=(2048, 32, low))
    assert err.max() <= TOL["fp32"]


def test_lowrank_wide_after_hyper_draw(bp, orc):  # noqa: F811
    K, t = 100, 3
    r = _sparse(2001, 15, 5)
    s = bp.Sampler(r, K, prec="fp32", seed=11)
    U0, V0 = (s.get_factor(side).astype(np.float64) for side in (bp.SIDE_U, bp.SIDE_V))
    s.sample_hyper(bp.SIDE_U, t)
    mu, Lam = s.get_hyper(bp.SIDE_U)
    s.update_side(bp.SIDE_U, t)
    got = s.get_factor(bp.SIDE_U).astype(np.float64)
    ch = orc.Chain(r.M, r.N, K, r.csr_ptr, r.csr_col, r.csr_val, r.test_row, r.test_col, r.test_val, seed=11)
    X = U0.copy()
    orc.update_rows(ch.csr_ptr, ch.csr_col, ch.csr_rc, V0, X, mu, Lam, 2.0, 11, orc.ROW_U, t)
    err = np.linalg.norm(got - X, axis=1) / np.maximum(np.linalg.norm(X, axis=1), 1e-3 * np.sqrt(K))
    assert err.max() <= TOL["fp32"]
    with pytest.raises(bp.BPMFError) as e:  # a plan by hand stays refused above K = 64
        s.set_plan(2048, 32, 8)
    assert e.value.code == bp.E_INVAL
    s.close()
