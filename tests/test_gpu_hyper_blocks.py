"""The hyperparameter draw at the edges of its 16 x 16 blocks (one component
below, at and above each block count it is built for) and of its row blocks
(fewer rows than one step of four, one block of 16 rows, one row more, many
blocks), against the oracle at the bar of the other hyper tests (1e-10)."""
import numpy as np
import pytest

import synth
from test_gpu_parity import HYPER_TOL, _random_state, bp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,K", [("fp32", 15), ("fp32", 16), ("fp32", 17), ("fp64", 33), ("fp32", 63), ("fp64", 64),
                                    ("fp32", 65), ("fp32", 80), ("fp32", 112), ("bf16", 113), ("fp32", 128)])
@pytest.mark.parametrize("M,N", [(3, 16), (17, 40001)])
def test_hyper_draw_blocks(bp, orc, prec, K, M, N):  # noqa: F811
    r = synth.random_small(6, M, N, 30, 2)
    s = bp.Sampler(r, K, prec=prec, seed=41)
    U, V, _, _ = _random_state(np.random.default_rng(K), M, N, K)
    s.set_factor(bp.SIDE_U, U)
    s.set_factor(bp.SIDE_V, V)
    for side, stream in ((bp.SIDE_U, orc.HYP_U), (bp.SIDE_V, orc.HYP_V)):
        s.sample_hyper(side, 4)
        mu, Lam = s.get_hyper(side)
        X = s.get_factor(side).astype(np.float64)
        mu_r, Lam_r = orc.hyper_draw(X, np.zeros(K), 2.0, float(K), np.eye(K), 41, stream, 4)
        assert np.allclose(Lam, Lam_r, rtol=HYPER_TOL, atol=HYPER_TOL * np.abs(Lam_r).max())
        assert np.allclose(mu, mu_r, rtol=HYPER_TOL, atol=HYPER_TOL * (1 + np.abs(mu_r).max()))
        assert np.array_equal(Lam, Lam.T)
    s.close()
