"""Multi-job launches with workgroups to spare: the jobs that end last take
more tiles; every job stays the oracle's, whatever the launch may hold."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("max_wgs", [0, 11, 16, 40])
def test_levelled_jobs_match_the_oracle(max_wgs):
    # unequal ends (800 last), equal ones (the two 400s), tile counts with
    # and without XCD bands, a job that no launch splits further (16)
    specs = [(400, 3, [1], 6), (800, 5, [1, 3], 5), (136, 3, [1], 3),
             (400, 5, [1, 3], 6), (16, 3, [1], 2), (400, 8, [1, 2, 5], 4)]
    ps, js, lats, g0s = [], [], [], []
    for i, (L, S, K, n) in enumerate(specs):
        p, j = pair(L, S, K, 0.5 + i, 1.0, 1.0, seed=70 + i, replica=i)
        ps.append(p)
        js.append(j)
        g0s.append(random_lattice(L, S, seed=i, domain=2))
        lats.append(dev(g0s[-1]))
    ps[0] = ps[0].with_launch(max_wgs=max_wgs)
    escg.step_batch(ps, lats, [7] * len(specs), [s[3] for s in specs])
    assert escg.last_route() == "persistent"
    for (L, S, K, n), j, g0, lat in zip(specs, js, g0s, lats):
        O.o2_run(j, g0, 7, n, want_counts=False)
        assert np.array_equal(host(lat), g0), (L, S)
    escg.async_status()
