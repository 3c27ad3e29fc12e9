"""Algorithm 1 takes its batch sizes as any iterable of integers: a range (not unrolled), a list, an array, an iterator."""
import numpy as np
import pytest

from paper_2211_13878_amd import alg1, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", [3, 8])
def test_batch_sizes_of_every_kind(window):
    model = workloads.Alg1Model(11, 19, 4, alg1.strategy_counts(4))
    want = None
    for sizes in (range(1, 10 ** 9), range(1, 400), list(range(1, 400)), np.arange(1, 400), iter(range(1, 400)), tuple(range(1, 400))):
        r = alg1.optimize(model, 4, 2300, sizes, window=window)
        got = (r.throughput, r.batch, r.pp, r.cost, r.plans, r.n_explored, r.stopped, r.c_p.tolist())
        want = want or got
        assert got == want and r.stopped and r.n_explored > window
    for sizes in (range(4, 4), [], range(2, 9, 3), [2, 5, 8]):
        r = alg1.optimize(model, 4, 2300, sizes, window=window)
        assert r.n_explored == len(sizes) and not r.stopped
