"""The patch kernel (escg_step_mcs on lattices of any even side) against the
oracle, byte for byte: every remainder of L mod 8, one to three quads a
thread, counts by the counting wave and by the updating waves, both species
classes, probabilities, both neighbourhoods, runs shorter and longer than the
MCS between two halo exchanges."""
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
    (72, 3, [1], 17, False, False),       # smallest, counting wave
    (90, 5, [1, 3], 9, False, False),     # smallest with a partial quad
    (92, 3, [1], 1, True, False),         # one MCS: no exchange
    (94, 7, [1, 2], 8, False, True),
    (100, 13, [1, 3], 7, False, False),   # histogram, counting wave
    (102, 1, [], 6, False, False),
    (300, 3, [1], 40, False, False),
    (404, 8, [1, 3], 7, True, True),
    (500, 3, [1], 13, False, False),
    (502, 5, [1, 3], 6, True, False),
    (1002, 3, [1], 5, False, False),
    (1202, 31, [1, 4, 9], 4, False, False),  # histogram by updating waves
    (1600, 5, [1, 3], 4, False, True),    # counts by the updating waves
    (2166, 4, [1], 3, False, False),      # two and three quads a thread
    (3190, 5, [1, 3], 2, False, False),
    (3200, 8, [1, 3], 2, False, False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{c[0]}_S{c[1]}")
def test_patches_bit_exact(case):
    L, S, K, n, moore, prob = case
    D = O.circulant_matrix(S, K) if K else np.zeros((S, S), np.uint8)
    P = probabilities(D, seed=L) if prob else None
    p, j = pair(L, S, None, 3e-5 * L * L / 2, seed=L + 5, replica=2, D=D,
                moore=moore, P=P, route="auto")
    g0 = random_lattice(L, S, seed=L, domain=3)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 1 << 20, n)
    for counts in (True, False):
        lat = dev(g0)
        cnt = torch.full(((n + 1) * (S + 1),), -1, dtype=torch.int32,
                         device="cuda:0") if counts else None
        escg.step_mcs(p, lat, 1 << 20, n, cnt)
        assert escg.last_route() == "persistent", escg.last_error()
        assert np.array_equal(host(lat), ref), counts
        if counts:
            assert np.array_equal(host(cnt).reshape(rc.shape), rc)
    lat = dev(g0)  # the same with the library's fixed scratch, in two calls
    cnt = torch.full((2 * (S + 1),), -1, dtype=torch.int32, device="cuda:0")
    if n > 1:
        escg.step_mcs_static(p, lat, 1 << 20, n - 1, None)
    escg.step_mcs_static(p, lat, (1 << 20) + n - 1, 1, cnt)
    assert np.array_equal(host(lat), ref)
    assert np.array_equal(host(cnt), rc[n - 1:].reshape(-1))
    escg.async_status()


def test_run_until_of_a_ragged_lattice_past_the_lds():
    D = np.array([[0, 1, 1], [0, 0, 0], [0, 0, 0]], np.uint8)
    p, j = pair(406, 3, None, 0.5, 1.0, 1.0, seed=3, D=D)
    g = j.init()
    lat = dev(g)
    res = torch.full((6,), -1, dtype=torch.int32, device="cuda:0")
    escg.run_until_extinction(p, lat, 0, 90, escg.STOP_FIRST_EXTINCTION, res)
    ref = O.o2_run_until(j, g, 0, 90, O.FIRST_EXTINCTION)
    assert np.array_equal(host(res), ref)
    assert np.array_equal(host(lat), g)


def test_ragged_lattice_under_capture_takes_an_ordinary_launch():
    """L % 8 != 0 in a captured graph: replayed with eager work between, each
    replay gives the eager bytes."""
    L, S, n = 100, 3, 3
    p, j = pair(L, S, [1], 1.5, seed=9, route="auto")
    g0 = random_lattice(L, S, seed=4, domain=2)
    ref = g0.copy()
    rc = O.o2_run(j, ref, 5, n)
    lat = dev(g0)
    cnt = torch.zeros((n + 1) * (S + 1), dtype=torch.int32, device="cuda:0")
    escg.step_mcs(p, lat, 5, n, cnt)
    assert escg.last_route() == "persistent"
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        escg.step_mcs(p, lat, 5, n, cnt)
    assert escg.last_route() == "lds"
    for _ in range(3):
        lat.copy_(dev(g0))
        cnt.zero_()
        graph.replay()
        assert np.array_equal(host(lat), ref)
        assert np.array_equal(host(cnt).reshape(rc.shape), rc)
        other = dev(g0)
        escg.step_mcs(p, other, 5, n, None)
        assert np.array_equal(host(other), ref)
