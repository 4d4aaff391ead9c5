"""The patch sweep (escg_step_mcs on lattices that the LDS of all CUs together
cannot hold) against the oracle, byte for byte: ragged and even quad rows,
runs that are no multiple of a launch's MCS, both species classes,
probabilities, both neighbourhoods, launches with more patches than
workgroups, and under capture."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair, probabilities

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [
    # L, S, K, n_mcs, moore, probabilities
    (3404, 3, [1], 5, False, False),      # two blocks in the last quad
    (3530, 7, [1, 2], 3, True, False),    # one block in the last quad
    (3902, 5, [1, 3], 4, False, True),    # three blocks in it
    (4102, 8, [1, 3], 2, True, True),     # histogram counts
    (5000, 13, [1, 3], 1, False, False),  # held by all CUs as uniform tiles
    (6008, 13, [1, 3], 1, False, False),  # no partial quad, one launch
    (6002, 4, [1], 3, False, False),      # several patches a workgroup
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{c[0]}_S{c[1]}")
def test_sweep_bit_exact(case):
    L, S, K, n, moore, prob = case
    D = O.circulant_matrix(S, K)
    P = probabilities(D, seed=L) if prob else None
    p, j = pair(L, S, None, 3e-5 * L * L / 2, seed=L + 5, replica=2, D=D,
                moore=moore, P=P, route="auto")
    g0 = random_lattice(L, S, seed=L, domain=3)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 1 << 20, n)
    route = "persistent" if L == 5000 else "tiled"
    for counts in (True, False):
        lat = dev(g0)
        cnt = torch.full(((n + 1) * (S + 1),), -1, dtype=torch.int32,
                         device="cuda:0") if counts else None
        escg.step_mcs(p, lat, 1 << 20, n, cnt)
        assert escg.last_route() == route, escg.last_error()
        assert np.array_equal(host(lat), ref), counts
        if counts:
            assert np.array_equal(host(cnt).reshape(rc.shape), rc)


def test_sweep_under_capture():
    L, S, n = 3406, 3, 4
    p, j = pair(L, S, [1], 90.0, seed=9, route="auto")
    g0 = random_lattice(L, S, seed=4, domain=2)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 5, n)
    lat = dev(g0)
    cnt = torch.zeros((n + 1) * (S + 1), dtype=torch.int32, device="cuda:0")
    escg.step_mcs(p, lat, 5, n, cnt)  # first use outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        escg.step_mcs(p, lat, 5, n, cnt)
    for _ in range(3):
        lat.copy_(dev(g0))
        cnt.zero_()
        graph.replay()
        assert np.array_equal(host(lat), ref)
        assert np.array_equal(host(cnt).reshape(rc.shape), rc)
        other = dev(g0)
        escg.step_mcs(p, other, 5, n, None)
        assert np.array_equal(host(other), ref)
