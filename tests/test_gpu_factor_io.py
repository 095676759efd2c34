"""Host copies of the factors (bpmf_get_factor / bpmf_set_factor) go through
2 MiB staging chunks: whole, ragged and several chunks, with and without row
padding (K mod 4) and degree-order relabelling."""
import numpy as np
import pytest

import paper_1705_04159_amd as bp
import synth

CHUNK = 2 << 20  # bytes of one staging chunk


@pytest.mark.gpu
@pytest.mark.parametrize("K,prec,rows", [
    (32, "fp32", CHUNK // 128), (32, "fp32", CHUNK // 128 + 1), (32, "bf16", 5 * (CHUNK // 128) // 2),
    (33, "fp32", CHUNK // 132), (33, "fp32", 3 * (CHUNK // 132) + 1), (1, "fp32", 7),
    (10, "fp64", CHUNK // 80 + 1), (64, "fp64", 2 * (CHUNK // 512)),
])
@pytest.mark.parametrize("reorder", [False, True])
def test_factor_round_trip(K, prec, rows, reorder):
    r = synth.random_small(5, rows, 11, 4000 if rows > 1000 else 20, 4)
    s = bp.Sampler(r, K, prec=prec, seed=3, reorder=reorder)
    X = np.random.default_rng(K).standard_normal((rows, K)).astype(s.dtype)
    s.set_factor(bp.SIDE_U, X)
    assert np.array_equal(s.get_factor(bp.SIDE_U), X)
    # the device sees the same rows: one-component products against V
    V = np.zeros((r.N, K), s.dtype)
    V[3, K - 1] = 1.0
    s.set_factor(bp.SIDE_V, V)
    pick = np.unique(np.linspace(0, rows - 1, 50).astype(np.int32))
    got = s.predict(pick, np.full(len(pick), 3, np.int32))
    want = (X[pick, K - 1].astype(np.float64) + s.mean_rating).astype(np.float32)
    assert np.array_equal(got, want)
    s.close()
