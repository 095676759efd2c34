"""The FP64 matrix-core row kernel at the edges of its tiles: every block
count, both sides of each 16-component boundary, a row a wavefront and (K <= 16,
many rows) four, split rows, rows without ratings.  Single steps against the oracle on identical inputs, at the FP64 bar
of the other parity tests (1e-12 a row)."""
import pytest

import synth
from test_gpu_parity import TOL, bp, single_step  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 15, 16, 17, 31, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("M,nnz,split", [(310, 9000, 0), (310, 24000, 257), (4703, 60011, 0), (4703, 60011, 300)])
def test_fp64_rows(bp, orc, K, M, nnz, split):  # noqa: F811
    r = synth.random_small(K, M, 91, nnz, 8, empty_rows=3)
    for side in (0, 1):
        err, _, _ = single_step(bp, orc, r, K, "fp64", side, split=split)
        assert err.max() <= TOL["fp64"]


# more than 10240 light rows: four to a wavefront up to K = 16, with a ragged
# last wavefront
@pytest.mark.parametrize("K", [1, 7, 16, 17])
@pytest.mark.parametrize("M,split", [(10243, 0), (10603, 0), (10603, 200)])
def test_fp64_many_rows(bp, orc, K, M, split):  # noqa: F811
    r = synth.random_small(K, M, 91, 90017, 8, empty_rows=3)
    for side in (0, 1):
        err, _, _ = single_step(bp, orc, r, K, "fp64", side, split=split)
        assert err.max() <= TOL["fp64"]
