"""The kernel with two copies of a lattice in LDS at the largest sides it takes
(280; 264 with more than seven species) and just past them, against the
oracle."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from tests.gpu_util import dev, host, pair
from tests.test_extinction_gpu import _batch, oracle_until

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,S,K", [(278, 3, [1]), (280, 5, [1, 3]),
                                   (282, 3, [1]), (262, 9, [1, 2, 4]),
                                   (264, 31, [1, 7]), (266, 9, [1, 2, 4])])
def test_largest_sides(L, S, K):
    p, j = pair(L, S, K, 3.0, seed=5, replica=L, route="lds")
    for mode, cap in ((escg.STOP_NONE, 5), (escg.STOP_FIRST_EXTINCTION, 7)):
        g = j.init()
        lat = dev(g)
        r = oracle_until(j, g, 3, cap, mode)
        res = torch.full((S + 3,), -1, dtype=torch.int32, device="cuda:0")
        escg.run_until_extinction(p, lat, 3, cap, mode, res)
        assert escg.last_route() == "lds"
        assert np.array_equal(host(res), r)
        assert np.array_equal(host(lat), g)
        lats, rr = _batch([(p, j, cap, None)], mode, True, [3])
        assert np.array_equal(rr[0][:S + 3], r)
        assert np.array_equal(lats[0], g)


@pytest.mark.parametrize("sides", [(2, 4, 8, 6), (10, 16, 2, 14), (24, 18, 8),
                                   (34, 30, 2), (46, 48, 64), (72, 70, 6)])
@pytest.mark.parametrize("S,K", [(3, [1]), (9, [1, 2, 4])])
def test_small_batches(sides, S, K):
    """Workgroups of as many waves as the largest lattice has quads for."""
    for mode in (escg.STOP_FIRST_EXTINCTION, escg.STOP_MONOCULTURE,
                 escg.STOP_NONE):
        jobs = []
        for i in range(3 * len(sides)):
            L = sides[i % len(sides)]
            p, j = pair(L, S, K, [0.5, 4.0, 0.0][i % 3], seed=5, replica=i,
                        moore=i % 2 == 1)
            jobs.append((p, j, [300, 40, 0, 1][i % 4], None))
        lats, r = _batch(jobs, mode, True, [i for i in range(len(jobs))])
        for i, ((p, j, cap, _), lat, rr) in enumerate(zip(jobs, lats, r)):
            g = j.init()
            want = oracle_until(j, g, i, cap, mode)
            assert np.array_equal(rr[:S + 3], want), (p.L, cap, rr, want)
            assert np.array_equal(lat, g), (p.L, cap)
