"""The generic row kernel, which factors of 1 GiB (2^21 users) and sides of 2^24
rows fall back to: both sides, rows without ratings, split movies, every
precision.  Single steps against the oracle at the bars of the other parity
tests, on the rated users and some others."""
import numpy as np
import pytest

import synth
from test_gpu_parity import TOL, _bf16_round, bp, row_errors  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,K,M", [("fp64", 64, 1 << 21), ("fp32", 128, 1 << 21), ("bf16", 127, 1 << 21),
                                      ("fp64", 2, (1 << 24) + 1), ("fp32", 3, 1 << 24)])
def test_beyond_the_matrix_core_kernels(bp, orc, prec, K, M):  # noqa: F811
    degrees = [0, 1, 2, 15, 16, 17, 31, 33, 100, 257, 1000, 2049, 5000, 9001]
    rng = np.random.default_rng(K)
    users = np.concatenate([rng.choice(M, d, replace=False) for d in degrees])
    movies = np.repeat(np.arange(len(degrees)), degrees)
    vals = (rng.standard_normal(len(users)) + 3.0).astype(np.float32)
    r = synth._assemble("gib", M, len(degrees), users, movies, vals, 0.0, rng, 8)
    A = rng.standard_normal((K, K))
    mu, Lam = rng.standard_normal(K) * 0.1, A @ A.T / K + np.eye(K)
    s = bp.Sampler(r, K, prec=prec, seed=21)
    ch = orc.Chain(r.M, r.N, K, r.csr_ptr, r.csr_col, r.csr_val, r.test_row, r.test_col, r.test_val, seed=21)

    def gathered(side):
        Y = s.get_factor(side).astype(np.float64)
        return _bf16_round(Y) if prec == "bf16" else Y

    rows = np.unique(np.concatenate([users[-400:], users[:300], np.arange(0, M, M // 300), [M - 1]]))
    s.set_hyper(bp.SIDE_U, mu, Lam)
    Y = gathered(bp.SIDE_V)
    s.update_side(bp.SIDE_U, 3)
    X = np.zeros((M, K))
    orc.update_rows(ch.csr_ptr, ch.csr_col, ch.csr_rc, Y, X, mu, Lam, 2.0, 21, orc.ROW_U, 3, rows=rows)
    err = row_errors(s.get_factor(bp.SIDE_U)[rows].astype(np.float64), X[rows])
    assert err.max() <= TOL[prec]
    del X
    s.set_hyper(bp.SIDE_V, mu, Lam)
    Y = gathered(bp.SIDE_U)
    s.update_side(bp.SIDE_V, 4)
    X = np.zeros((r.N, K))
    orc.update_rows(ch.csc_ptr, ch.csc_row, ch.csc_rc, Y, X, mu, Lam, 2.0, 21, orc.ROW_V, 4)
    err = row_errors(s.get_factor(bp.SIDE_V).astype(np.float64), X)
    assert err.max() <= TOL[prec]
    s.close()
