"""Launch choices that a caller names, each against the oracle: workgroup sizes
and workgroups per CU of a batch, tile shapes of a multi-job launch, and the
equal-tile persistent kernel (steps and runs until extinction), which also
takes single lattices past the patches' size by itself."""
import functools

import numpy as np
import pytest

import oracle as O
from paper_2508_16639_amd import escg
from paper_2508_16639_amd.workloads import random_lattice
from tests.gpu_util import dev, host, pair, probabilities
from tests.test_extinction_gpu import (D_TAKEOVER, MODES, _batch,
                                       oracle_until)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@functools.lru_cache(maxsize=None)
def batch_reference(kind, mode):
    jobs, refs = [], []
    for i, L in enumerate([64, 96, 130, 192, 256, 250, 10, 90]):
        S, K = (9, [1, 2, 4]) if kind == "wide" and i % 2 else (3, [1])
        D = O.circulant_matrix(S, K)
        P = probabilities(D, seed=L) if kind == "prob" and i % 2 else None
        p, j = pair(L, S, None, 2.0, seed=9, replica=i, D=D, moore=i % 3 == 2,
                    P=P, route="auto")
        cap = [40, 33, 5, 17][i % 4]
        g = j.init()
        refs.append((oracle_until(j, g, 3 * i, cap, mode), g))
        jobs.append((p, j, cap, None))
    return jobs, refs


@pytest.mark.parametrize("kind", ["plain", "wide", "prob"])
@pytest.mark.parametrize("threads,wg_per_cu", [
    (128, 0), (256, 1), (256, 2), (384, 0), (512, 1), (512, 2), (0, 1),
    (1024, 0)])
def test_batch_workgroups(kind, threads, wg_per_cu):
    for mode in MODES:
        jobs, refs = batch_reference(kind, mode)
        p0 = jobs[0][0].with_launch(threads=threads, wg_per_cu=wg_per_cu)
        lats, r = _batch([(p0,) + jobs[0][1:]] + jobs[1:], mode, True,
                         [3 * i for i in range(len(jobs))])
        for (p, _, _, _), lat, rr, (want, g) in zip(jobs, lats, r, refs):
            assert np.array_equal(rr[:p.S + 3], want), (p.L, mode)
            assert (rr[p.S + 3:] == 0).all()
            assert np.array_equal(lat, g), (p.L, mode)


@pytest.mark.parametrize("S,moore,prob", [(5, False, False), (5, True, False),
                                          (7, False, True), (13, True, True),
                                          (9, False, False)])
@pytest.mark.parametrize("shapes", [((100, 400), (200, 400)),
                                    ((200, 200), (160, 160)),
                                    ((40, 80), (100, 200))])
def test_multi_job_tile_shapes(S, moore, prob, shapes):
    ps, lats, gs = [], [], []
    for i, (L, tile) in enumerate(zip((400, 800), shapes)):
        D = O.circulant_matrix(S, [1, 3])
        P = probabilities(D, seed=L) if prob else None
        p, j = pair(L, S, None, 5.0, seed=4, replica=i, D=D, moore=moore, P=P,
                    route="auto")
        ps.append(p.with_launch(tile=tile))
        g = random_lattice(L, S, seed=L, domain=2)
        lats.append(dev(g))
        O.o2_run(j, g, 5, 3 + i, want_counts=False)
        gs.append(g)
    escg.step_batch(ps, lats, [5, 5], [3, 4])
    assert escg.last_route() == "persistent"
    for lat, g in zip(lats, gs):
        assert np.array_equal(host(lat), g)
    escg.async_status()


@functools.lru_cache(maxsize=None)
def step_reference(L, S, moore, prob, n):
    D = O.circulant_matrix(S, [1, 2, 5] if S > 7 else [1, 3])
    P = probabilities(D, seed=S) if prob else None
    p, j = pair(L, S, None, 51.2, seed=17, replica=1, D=D, moore=moore, P=P,
                route="auto")
    g0 = random_lattice(L, S, seed=S + 1, domain=5)
    ref = g0.copy()
    return p, g0, ref, O.o2_run(j, ref, 3, n)


@pytest.mark.parametrize("S", [5, 13])
@pytest.mark.parametrize("moore,prob", [(False, False), (True, False),
                                        (False, True), (True, True)])
@pytest.mark.parametrize("L,tile,threads", [
    (3200, (100, 400), 0), (3200, (160, 320), 0), (3200, (200, 200), 512),
    (3600, None, 0)])
def test_equal_tiles(S, moore, prob, L, tile, threads):
    """Named shapes (list walk, column walk, fewer threads) and the kernel
    that a side of 3600 takes by itself."""
    n = 2
    p, g0, ref, rc = step_reference(L, S, moore, prob, n)
    q = p.with_launch(tile=tile, threads=threads)
    assert escg.tile_plan(q, True) is not None
    lat = dev(g0)
    cnt = torch.full(((n + 1) * (S + 1),), -1, dtype=torch.int32,
                     device="cuda:0")
    escg.step_mcs(q, lat, 3, n, cnt)
    assert escg.last_route() == "persistent"
    assert np.array_equal(host(lat), ref)
    assert np.array_equal(host(cnt).reshape(rc.shape), rc)
    escg.async_status()


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("L,tile,sel,moore,prob", [
    (80, (16, 40), 1.0, False, False), (80, (8, 16), 0.03, True, False),
    (96, (48, 48), 0.05, False, True), (416, (104, 104), 1.0, False, False)])
def test_run_until_on_equal_tiles(mode, L, tile, sel, moore, prob):
    P = 0.9 * D_TAKEOVER if prob else None
    p, j = pair(L, 3, None, 0.5, sel, 1.0, seed=77, replica=1, D=D_TAKEOVER,
                moore=moore, P=P, route="auto")
    p = p.with_launch(tile=tile)
    cap = 150 if mode == escg.STOP_NONE or L > 400 else 3000
    g = j.init()
    lat = dev(g)
    res = torch.full((6,), -1, dtype=torch.int32, device="cuda:0")
    escg.run_until_extinction(p, lat, 5, cap, mode, res)
    assert escg.last_route() == "persistent"
    want = oracle_until(j, g, 5, cap, mode)
    assert np.array_equal(host(res), want)
    assert np.array_equal(host(lat), g)
