"""Plans above K = 64, where the rank-one path follows the library's rule: what
autotune returns is taken back by set_plan and gives the same plan, no candidate
is tried twice, and a cut-off by hand is refused.  Up to K = 64 a cut-off of 0
leaves no row on the path, rows without ratings included."""
import numpy as np
import pytest

import synth
from test_gpu_lowrank_wide import _sparse
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


def test_autotuned_plan_round_trip(bp, orc):  # noqa: F811
    r = _sparse(9001, 300, 7)
    s = bp.Sampler(r, 100, prec="fp32", seed=3)
    n = s.lowrank_rows(bp.SIDE_U)
    assert n == (np.diff(r.csr_ptr) <= 8).sum()
    split, kmax, low, tried = s.autotune(1)
    plans = [t[:3] for t in tried]
    assert len(set(plans)) == len(plans) and (split, kmax, low) in plans and {p[2] for p in plans} == {0}
    assert s.lowrank_rows(bp.SIDE_U) == n
    before = s.get_plan(bp.SIDE_V)
    s.set_plan(split, kmax, low)
    assert s.lowrank_rows(bp.SIDE_U) == n
    for a, b in zip(before, s.get_plan(bp.SIDE_V)):
        assert np.array_equal(a, b)
    for dmax in (4, 8, 16):
        with pytest.raises(bp.BPMFError) as e:
            s.set_plan(split, kmax, dmax)
        assert e.value.code == bp.E_INVAL
    assert s.lowrank_rows(bp.SIDE_U) == n
    s.close()
    rows = np.arange(0, r.M, 11)
    err, _, _ = single_step(bp, orc, r, 100, "fp32", bp.SIDE_U, rows=rows, plan=(split, kmax, low))
    assert err.max() <= TOL["fp32"]


@pytest.mark.parametrize("K", [16, 48, 100])
def test_cutoff_0_means_off(bp, orc, K):  # noqa: F811
    r = synth.random_small(11, 1003, 150, 9000, 10, empty_rows=20)
    s = bp.Sampler(r, K, prec="fp32", seed=1)
    s.set_plan(256, 32, 0)
    assert s.lowrank_rows(bp.SIDE_U) == 0 and s.lowrank_rows(bp.SIDE_V) == 0
    s.close()
    for side in (bp.SIDE_U, bp.SIDE_V):
        err, _, _ = single_step(bp, orc, r, K, "fp32", side, plan=(256, 32, 0))
        assert err.max() <= TOL["fp32"]
