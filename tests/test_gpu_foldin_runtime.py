"""Fold-in serving is refused, before any of its GPU work, in a process that runs
on an older HIP runtime than the library was built for (one that loaded PyTorch
first runs on PyTorch's)."""
import subprocess
import sys
from pathlib import Path

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import torch
torch.cuda.init()
import paper_1705_04159_amd as bp
import synth
if tuple(int(x) for x in torch.version.hip.split(".")[:2]) >= (7, 2):
    print("same runtime")
    raise SystemExit
s = bp.Sampler(synth.random_small(7, 40, 30, 300, 8), 8, prec="fp32", seed=3)
try:
    s.store_sample()
except bp.BPMFError as e:
    print("refused:", e)
s.close()
"""


def test_refused_on_an_older_runtime():
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=Path(__file__).resolve().parent.parent,
                       capture_output=True, text=True, timeout=110)
    assert p.returncode == 0, p.stderr
    if "same runtime" in p.stdout:
        pytest.skip("PyTorch brings the runtime that the library was built for")
    assert "refused:" in p.stdout and "older HIP runtime" in p.stdout
