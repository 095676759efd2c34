"""Predictions of caller pairs on both sides of the limit up to which the kernel
reads them in place (349,525 pairs) and of its blocks of 64 and 256 pairs, against
the allocation-free entry point, bit for bit, and numpy."""
import numpy as np
import pytest

import paper_1705_04159_amd as bp
import synth

LIMIT = 2 * (2 << 20) // 12


@pytest.mark.gpu
@pytest.mark.parametrize("prec,K", [("fp32", 32), ("fp32", 37), ("fp64", 10), ("bf16", 100)])
@pytest.mark.parametrize("reorder", [False, True])
def test_predict_pairs_sizes(prec, K, reorder):
    r = synth.random_small(7, 1003, 811, 9000, 6)
    s = bp.Sampler(r, K, prec=prec, seed=9, reorder=reorder)
    U, V = (s.get_factor(side).astype(np.float64) for side in (bp.SIDE_U, bp.SIDE_V))
    rng = np.random.default_rng(K)
    for n in (1, 3, 63, 64, 65, 255, 257, 20000, LIMIT, LIMIT + 1):
        row, col = (rng.integers(0, m, n).astype(np.int32) for m in (r.M, r.N))
        got = s.predict(row, col)
        assert np.array_equal(got, s.predict_noalloc(row, col))
        want = (U[row] * V[col]).sum(1) + s.mean_rating
        assert np.abs(got - want).max() <= K * 2.0 ** -23 * (1 + np.abs(want).max())
    for bad in ((-1, 0), (r.M, 0), (0, -5), (0, r.N)):
        row, col = np.zeros(70, np.int32), np.zeros(70, np.int32)
        row[66], col[66] = bad
        with pytest.raises(bp.BPMFError) as e:
            s.predict(row, col)
        assert e.value.code == bp.E_RANGE
    s.close()
