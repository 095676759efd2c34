"""The blocked kernel's split rows with segments too short to be dealt to four
wavefronts (one-wave workgroups), beside whole rows that are and are not, at
seven and eight blocks of components: against the oracle at the bars of the
other single steps."""
import pytest

from test_gpu_heavy_rows import DEGREES, _columns
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,K", [("fp32", 112), ("fp32", 113), ("fp32", 128), ("bf16", 113), ("bf16", 128)])
@pytest.mark.parametrize("split", [130, 255, 300, 512])
def test_short_segments(bp, orc, prec, K, split):  # noqa: F811
    r = _columns(DEGREES, 3000, K)
    err, _, _ = single_step(bp, orc, r, K, prec, 1, split=split)
    assert err.max() <= TOL[prec]


@pytest.mark.parametrize("prec,K", [("fp32", 48), ("fp32", 128), ("bf16", 17), ("bf16", 128)])
def test_light_rows_only(bp, orc, prec, K):  # noqa: F811
    r = _columns([0, 1, 31, 32, 33, 64, 65, 255, 256] * 40, 1500, K)
    err, _, _ = single_step(bp, orc, r, K, prec, 1)
    assert err.max() <= TOL[prec]
