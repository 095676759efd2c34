"""Reads of one context's state from several threads at a time (factors of more
than one staging chunk, hyperparameters, predictions of pairs below and above
the number that is read in place) give what each gives alone."""
import threading

import numpy as np
import pytest

import paper_1705_04159_amd as bp
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,K,reorder", [("fp32", 33, False), ("fp64", 64, True)])
def test_concurrent_reads(prec, K, reorder):
    r = synth.random_small(30, 20011, 3001, 60000, 6)
    s = bp.Sampler(r, K, prec=prec, seed=8, reorder=reorder)
    for side in (bp.SIDE_V, bp.SIDE_U):
        s.sample_hyper(side, 1)
        s.update_side(side, 1)
    rng = np.random.default_rng(3)
    calls = [lambda side=side: (s.get_factor(side),) for side in (bp.SIDE_U, bp.SIDE_V)]
    calls += [lambda side=side: s.get_hyper(side) for side in (bp.SIDE_U, bp.SIDE_V)]
    for n in (1, 70, 20000, 300000, 360000):
        row, col = (rng.integers(0, m, n).astype(np.int32) for m in (r.M, r.N))
        calls.append(lambda row=row, col=col: (s.predict(row, col),))
    alone = [f() for f in calls]
    wrong = []

    def work(k):
        try:
            for _ in range(30):
                if not all(np.array_equal(a, b) for a, b in zip(calls[k](), alone[k])):
                    wrong.append(k)
        except Exception as e:  # noqa: BLE001 -- reported below
            wrong.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    s.close()
