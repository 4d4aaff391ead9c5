"""The kernel that keeps two copies of a lattice in one workgroup's LDS
(escg_batch_run's larger jobs, runs until extinction on the LDS route) against
the oracle: one to five quads a thread, every remainder of L mod 8, stops
found between two tests of the condition, at them, in the first MCS and not
at all, both species classes."""
import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair, probabilities
from tests.test_extinction_gpu import _batch, oracle_until

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

D_TAKEOVER = np.array([[0, 1, 1], [0, 0, 0], [0, 0, 0]], np.uint8)
MODES = [escg.STOP_FIRST_EXTINCTION, escg.STOP_MONOCULTURE, escg.STOP_NONE]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("L", [90, 100, 126, 182, 222])
def test_run_until_stops_exactly(L, mode):
    p, j = pair(L, 3, None, 0.5, 1.0, 1.0, seed=5, replica=L, D=D_TAKEOVER,
                route="lds")
    g0 = j.init()
    full = oracle_until(j, g0.copy(), 3, 140, mode)
    t = int(full[1])
    for cap in sorted({0, 1, 32, 33, max(t - 1, 0), t, t + 1, 140}):
        ref = g0.copy()
        r = oracle_until(j, ref, 3, cap, mode)
        lat = dev(g0)
        res = torch.full((6,), -1, dtype=torch.int32, device="cuda:0")
        escg.run_until_extinction(p, lat, 3, cap, mode, res)
        assert escg.last_route() == "lds"
        assert np.array_equal(host(res), r), (cap, host(res), r)
        assert np.array_equal(host(lat), ref), cap


@pytest.mark.parametrize("init", [True, False])
@pytest.mark.parametrize("wide", [False, True])
def test_batch_of_larger_lattices(init, wide):
    jobs = []
    for i, L in enumerate([90, 94, 128, 152, 184, 200, 226, 250, 254, 2, 30]
                          + ([] if wide else [268, 276])):
        S, K = ((9, [1, 2, 4]) if wide and i % 2 else (3, [1]))
        D = O.circulant_matrix(S, K)
        P = probabilities(D, seed=L) if i % 4 == 1 else None
        p, j = pair(L, S, None, 10.0 ** (i % 3), seed=50 + i, replica=i, D=D,
                    moore=i % 3 == 2, P=P)
        cap = [40, 33, 5, 64, 1, 0][i % 6]
        g0 = None if init else random_lattice(L, S, seed=i, domain=2)
        jobs.append((p, j, cap, g0))
    lats, r = _batch(jobs, escg.STOP_FIRST_EXTINCTION, init,
                     [7 * i for i in range(len(jobs))])
    for i, ((p, j, cap, g0), lat, rr) in enumerate(zip(jobs, lats, r)):
        g = j.init() if init else g0.copy()
        ref = oracle_until(j, g, 7 * i, cap, escg.STOP_FIRST_EXTINCTION)
        assert np.array_equal(rr[:p.S + 3], ref), (p.L, rr, ref)
        assert (rr[p.S + 3:] == 0).all()
        assert np.array_equal(lat, g), p.L


def test_batch_kernels_agree():
    """The same batch by both kernels (a workgroup size asked for selects the
    one that updates in place), in every stop mode."""
    for mode in MODES:
        outs = []
        for kw in ({}, {"threads": 512}):
            jobs = []
            for i in range(24):
                L = [96, 130, 176, 256][i % 4]
                p, j = pair(L, 3, None, 0.4, 1.0, 1.0, seed=2, replica=i,
                            D=D_TAKEOVER)
                jobs.append((p.with_launch(**kw), j, 120, None))
            lats, r = _batch(jobs, mode, True)
            outs.append((np.concatenate(lats), r))
        assert np.array_equal(outs[0][0], outs[1][0])
        assert np.array_equal(outs[0][1], outs[1][1])
