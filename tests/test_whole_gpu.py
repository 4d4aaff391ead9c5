"""The small-lattice kernel (one workgroup, one quad a thread: L <= 88 on the
LDS route) against the oracle, byte for byte: steps with and without counts,
runs until extinction and monoculture that stop at once, within and at the
end of their budget, and under capture."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair, probabilities
from tests.test_extinction_gpu import oracle_until

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("L,S,K,n,moore,prob", [
    (2, 3, [1], 70, False, False), (6, 8, [1, 3], 9, True, False),
    (8, 5, [1, 3], 130, False, False), (18, 7, [1, 2], 65, False, True),
    (64, 3, [1], 64, False, False), (66, 31, [1, 4], 5, False, False),
    (70, 13, [1, 3], 6, True, True), (88, 5, [1, 3], 5, False, False),
    (86, 4, [1], 0, False, False)])
def test_step_bit_exact(L, S, K, n, moore, prob):
    D = O.circulant_matrix(S, K)
    P = probabilities(D, seed=L) if prob else None
    p, j = pair(L, S, None, 0.7, seed=L, replica=1, D=D, moore=moore, P=P,
                route="lds")
    g0 = random_lattice(L, S, seed=L, domain=2)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 77, n)
    for counts in (True, False):
        lat = dev(g0)
        cnt = torch.full(((n + 1) * (S + 1),), -1, dtype=torch.int32,
                         device="cuda:0") if counts else None
        escg.step_mcs(p, lat, 77, n, cnt)
        assert np.array_equal(host(lat), ref)
        if counts:
            assert np.array_equal(host(cnt).reshape(rc.shape), rc)


D_TAKEOVER = np.array([[0, 1, 1], [0, 0, 0], [0, 0, 0]], np.uint8)


@pytest.mark.parametrize("mode", [escg.STOP_FIRST_EXTINCTION,
                                  escg.STOP_MONOCULTURE, escg.STOP_NONE])
@pytest.mark.parametrize("L", [2, 10, 30, 64, 70, 86])
def test_run_until_stops_exactly(L, mode):
    p, j = pair(L, 3, None, 0.5, 1.0, 1.0, seed=5, replica=L, D=D_TAKEOVER,
                route="lds")
    g0 = j.init()
    full = oracle_until(j, g0.copy(), 3, 400, mode)
    t = int(full[1])
    for cap in {0, 1, max(t - 1, 0), t, t + 1, 400}:
        ref = g0.copy()
        r = oracle_until(j, ref, 3, cap, mode)
        lat = dev(g0)
        res = torch.full((6,), -1, dtype=torch.int32, device="cuda:0")
        escg.run_until_extinction(p, lat, 3, cap, mode, res)
        assert np.array_equal(host(res), r), (cap, host(res), r)
        assert np.array_equal(host(lat), ref), cap
