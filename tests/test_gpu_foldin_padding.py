"""Fold-in at K mod 4 != 0, where a drawn factor's row ends in padding that the
score multiplies, on device memory that earlier owners left full of NaN and
infinity bits (as ids of -1 do), and the top-n selection with a mean that is the
NaN of all ones: against the oracle at the bars of the other fold-in tests."""
import ctypes

import numpy as np
import pytest

import synth
from test_gpu_foldin import _check_against_oracle, _wait, bp  # noqa: F401

pytestmark = pytest.mark.gpu

BATCH = 64  # requests that one batch's draws are allocated for


def _soil(sizes, words):
    """Device memory blocks of the given bytes, filled with `words` and freed."""
    hip = ctypes.CDLL("libamdhip64.so.7")  # the library's own HIP runtime
    hip.hipMalloc.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    hip.hipMemsetD32.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t]
    hip.hipFree.argtypes = [ctypes.c_void_p]
    held = []
    for n, size in enumerate(sizes):
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), size) == 0
        assert hip.hipMemsetD32(p, ctypes.c_int32(words[n % len(words)]).value, size // 4) == 0
        held.append(p)
    assert hip.hipDeviceSynchronize() == 0
    for p in held:
        assert hip.hipFree(p) == 0


@pytest.mark.parametrize("K,S", [(1, 3), (6, 16), (26, 10), (33, 9), (61, 2)])
def test_foldin_on_soiled_memory(bp, orc, K, S):  # noqa: F811
    r = synth.random_small(27, 400, 1853, 9000, min(K, 12))
    seed = 19
    s = bp.Sampler(r, K, prec="fp32", seed=seed, foldin_S=S)
    ld = (K + 3) // 4 * 4
    store = []
    for t in range(1, S + 1):
        for side in (bp.SIDE_V, bp.SIDE_U):
            s.sample_hyper(side, t)
            s.update_side(side, t)
        if t == 1:  # the first stored sample allocates the batches' buffers
            _soil([BATCH * S * ld * 4] * 24, [-1, 0x7F800000])
        s.store_sample()
        mu, Lam = s.get_hyper(bp.SIDE_U)
        store.append((s.get_factor(bp.SIDE_V).astype(np.float64), mu, Lam))
    rng = np.random.default_rng(K)
    reqs = []
    for n, top in ((0, 40), (3, 100), (700, 1), (1853, 5), (55, 64)):
        movie = rng.choice(r.N, n, replace=False).astype(np.int32)
        rating = rng.normal(3.0, 1.0, n).astype(np.float32)
        reqs.append((movie, rating, s.foldin_submit(movie, rating, top), top))
    for movie, rating, rid, top in reqs:
        _check_against_oracle(orc, s, store, movie, rating, rid, _wait(s, rid, top), top, seed)
    s.close()


@pytest.mark.parametrize("bits", [0xFFFFFFFF, 0xFFFFFFFE, 0x7FC00000])
def test_topn_with_a_nan_mean(bp, bits):  # noqa: F811
    """Every unrated movie is returned once when all are asked for, the one
    whose factor row is NaN among them."""
    r = synth.random_small(28, 100, 90, 1500, 6)
    s = bp.Sampler(r, 6, prec="fp32", seed=4, foldin_S=2)
    V = s.get_factor(bp.SIDE_V)
    V[17] = np.array(bits, np.uint32).view(np.float32)
    s.set_factor(bp.SIDE_V, V)
    s.store_sample()
    movie = np.array([3, 40, 88], np.int32)
    ids, mean, _, _ = _wait(s, s.foldin_submit(movie, np.array([1.0, 2.0, 4.0], np.float32), 90), 90)
    assert np.array_equal(np.sort(ids[:87]), np.setdiff1d(np.arange(90), movie))
    assert np.all(ids[87:] == -1)
    assert np.array_equal(np.isnan(mean[:87]), ids[:87] == 17)
    s.close()
