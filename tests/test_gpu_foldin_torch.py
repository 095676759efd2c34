"""Fold-in serving in a process that loaded PyTorch first and so runs on PyTorch's
HIP runtime: contexts made one after the other on the memory of those before
(26 components, a padded row of 28), against the oracle at the bars of the other
fold-in tests."""
import subprocess
import sys
from pathlib import Path

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import sys
import torch
torch.cuda.init()
sys.path.insert(0, "tests")
import numpy as np
import oracle
import paper_1705_04159_amd as bp
import synth
from test_gpu_foldin import _check_against_oracle, _wait
oracle.build()
for seed, (N, K, S) in enumerate([(2000, 32, 10), (18538, 26, 10), (18538, 26, 10)]):
    print("N", N, "K", K, "S", S, flush=True)
    r = synth.random_small(29, 500, N, 20000, 8)
    s = bp.Sampler(r, K, prec="fp32", seed=seed, foldin_S=S)
    store = []
    for t in range(1, S + 1):
        for side in (bp.SIDE_V, bp.SIDE_U):
            s.sample_hyper(side, t)
            s.update_side(side, t)
        s.store_sample()
        mu, Lam = s.get_hyper(bp.SIDE_U)
        store.append((s.get_factor(bp.SIDE_V).astype(np.float64), mu, Lam))
    rng = np.random.default_rng(seed)
    reqs = []
    for n in (20, 600):
        movie = rng.choice(N, n, replace=False).astype(np.int32)
        rating = rng.normal(3.0, 1.0, n).astype(np.float32)
        reqs.append((movie, rating, s.foldin_submit(movie, rating, 100)))
    for movie, rating, rid in reqs:
        _check_against_oracle(oracle, s, store, movie, rating, rid, _wait(s, rid, 100), 100, seed)
    s.close()
print("served")
"""


def test_foldin_after_torch():
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=Path(__file__).resolve().parent.parent,
                       capture_output=True, text=True, timeout=110)
    assert p.returncode == 0 and "served" in p.stdout, p.stdout + p.stderr
