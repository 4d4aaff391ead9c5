"""The work that is timed: what users of this library have it do, through its
public entry points, over the sizes and options they use.

Five kinds of work (``case["kind"]``):

* ``step``   one ``step_mcs`` call of ``mcs`` MCS with per-MCS counts on a
  lattice that the program holds and steps on and on (the command line's
  loop, an interactive viewer);
* ``sim``    a whole simulation: ``init``, then ``step_mcs`` with counts;
* ``until``  ``init``, then ``run_until_extinction`` (its host loop included);
* ``batch``  ``batch_run``: ``n`` replicas, each initialised and run to its
  first extinction or 20 L MCS;
* ``multi``  ``step_batch``: ``n`` lattices advanced together, as the job
  server does with its large jobs.

``L`` is the lattice side (the largest of a batch, the smallest of a multi),
``M`` the mobility, ``S`` the species of a circulant game, ``moore`` the 8-way
neighbourhood, ``prob`` dominance with win probabilities.
"""
import math

import numpy as np
import torch

from paper_2508_16639_amd import escg, workloads

# Site-updates of the largest drawn case (the largest listed one has 1.1e10).
DRAW_UPDATES = 2.0e9


def _case(name, kind, L, S, M, mcs, n=1, moore=False, prob=False):
    return {"name": name, "kind": kind, "L": L, "S": S, "M": M, "mcs": mcs,
            "n": n, "moore": moore, "prob": prob}


def listed():
    return [
        # the smallest call: a viewer that steps one MCS a frame
        _case("step_L64_1", "step", 64, 3, 1e-4, 1),
        # the small rock-paper-scissors workload (eps = 0.5), whole
        _case("sim_L64_100", "sim", 64, 3, 2 * 0.5 / 64**2, 100),
        # the command line's defaults: L = 200, M = 3e-5, 200 MCS a print
        _case("step_L200_200", "step", 200, 3, 3e-5, 200),
        # two sides of the paper's runtime table (100, 200, ... 800) that are
        # no multiple of 8: one that fits a workgroup's LDS, one that does not
        _case("step_L300_200", "step", 300, 3, 3e-5, 200),
        _case("step_L500_200", "step", 500, 3, 3e-5, 200),
        # the mid-size workload of the benchmark, a fifth of its MCS
        _case("sim_L512_2000", "sim", 512, 3, 1e-4, 2000),
        # the benchmark's headline: rock-paper-scissors-lizard-Spock
        _case("sim_L3200_1000", "sim", 3200, 5, 1e-5, 1000),
        # eight species, 8-way neighbourhood, win probabilities (the
        # replication of Park, Chen and Szolnoki)
        _case("step_L400_S8_200", "step", 400, 8, 3e-5, 200, moore=True,
              prob=True),
        # a lattice far too large for the chip's LDS
        _case("sim_L16384_8", "sim", 16384, 5, 1e-7, 8),
        # one extinction experiment (Reichenbach's), mobility near critical
        _case("until_L192", "until", 192, 3, 5e-4, 20 * 192),
        # a quarter of the benchmark's replica table
        _case("batch_1024", "batch", 256, 3, 0.0, 20 * 256, n=1024),
        # the server's large jobs, one iteration: L = 400, 800, 1600
        _case("multi_24", "multi", 400, 5, 1e-5, 500, n=24),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: sides of any parity of L / 2 over the whole
    range of each kind, any number of species, both neighbourhoods."""
    kind = rng.choice(["step", "step", "step", "sim", "sim", "until", "batch",
                       "multi"])
    S = rng.choice([3, 3, 4, 5, 5, 7, 8, 13])
    M = math.exp(rng.uniform(math.log(1e-6), math.log(1e-3)))
    moore, prob, n = rng.random() < 0.25, rng.random() < 0.2, 1
    if kind == "batch":
        L, n = 2 * _logint(rng, 24, 150), _logint(rng, 16, 512)
        mcs = 20 * L
        S, moore, prob = rng.choice([3, 5]), False, False
    elif kind == "multi":
        L, n = 8 * _logint(rng, 10, 60), rng.randint(2, 24)
        mcs = _logint(rng, 20, 500)
    elif kind == "until":
        L = 2 * _logint(rng, 16, 200)
        mcs = 20 * L
    else:
        L = 2 * _logint(rng, 8, 6000)
        mcs = _logint(rng, 1, 2000)
    per_mcs = (5.6 * n * L * L if kind == "multi" else
               0.47 * n * L * L if kind == "batch" else L * L)
    mcs = max(1, min(mcs, int(DRAW_UPDATES / per_mcs)))
    c = _case("", kind, L, S, M, mcs, n, moore, prob)
    del c["name"]
    return c


def _dominance(S):
    """Circulant offsets of a case: {1}, or {1, 3} from five species on."""
    return (1,) if S < 5 else (1, 3)


def _probabilities(S):
    """Win probabilities of a `prob` case (used where a dominates b)."""
    a = np.arange(S)
    return 0.3 + 0.6 * ((7 * a[:, None] + 3 * a[None, :]) % 11) / 10.0


def _params(c, seed, L=None, S=None, replica=0, M=None):
    L, S = L or c["L"], S or c["S"]
    M = c["M"] if M is None else M
    return escg.Params(L=L, S=S, dom=escg.circulant_dom(S, _dominance(S)),
                       ex=workloads.eps_from_mobility(M, L), sel=1.0, rep=1.0,
                       seed=seed, replica=replica, moore=c["moore"],
                       prob=_probabilities(S) if c["prob"] else None)


def _batch_table(c):
    """Sides and mobilities of the replicas: four sides up to L, mobility
    log-uniform on 1e-6 .. 1e-3, as the benchmark's table."""
    L = c["L"]
    sizes = tuple(max(2, 2 * (k * L // 8)) for k in (1, 2, 3, 4))
    return workloads.batch_replicas(c["n"], sizes=sizes)


def _multi_table(c):
    """(L, S, MCS) of each job: sides L, 2 L, 4 L in turn, three species and
    five (or the case's), each MCS count cut to 1e9 site-updates."""
    out = []
    for j in range(c["n"]):
        L = c["L"] << (j % 3)
        S = 3 if j % 2 == 0 else c["S"]
        out.append((L, S, max(1, min(c["mcs"], int(1e9 / (L * L))))))
    return out


def _lattice(L, S, seed):
    """The lattice a program holds: i.i.d. uniform sites in 2 x 2 patches,
    so that neighbours agree as often as in a running game."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randint(0, S + 1, (L // 2, L // 2), generator=g, device="cuda",
                      dtype=torch.uint8)
    return h.repeat_interleave(2, 0).repeat_interleave(2, 1).reshape(-1)


def prepare(case, seed):
    c, kind = case, case["kind"]
    i32 = dict(dtype=torch.int32, device="cuda")
    u8 = dict(dtype=torch.uint8, device="cuda")
    st = {"kind": kind, "case": c, "t": 0}
    if kind == "batch":
        tab = _batch_table(c)
        st["params"] = [_params(c, seed, L=int(tab.L[r]), replica=r,
                                M=float(tab.M[r])) for r in range(c["n"])]
        ends = np.cumsum(tab.L.astype(np.int64) ** 2 + 3 & ~3)
        st["offsets"] = np.concatenate([[0], ends[:-1]])
        st["max_mcs"] = np.minimum(tab.max_mcs, c["mcs"])
        st["lat"] = torch.zeros(int(ends[-1]), **u8)
        st["res"] = torch.zeros(c["n"] * escg.BATCH_RESULT_WORDS, **i32)
    elif kind == "multi":
        tab = _multi_table(c)
        st["params"] = [_params(c, seed + j, L=L, S=S)
                        for j, (L, S, _) in enumerate(tab)]
        st["lats"] = [_lattice(L, S, seed + j)
                      for j, (L, S, _) in enumerate(tab)]
        st["n_mcs"] = [n for _, _, n in tab]
    else:
        L, S = c["L"], c["S"]
        st["p"] = _params(c, seed)
        st["lat"] = (_lattice(L, S, seed) if kind == "step"
                     else torch.empty(L * L, **u8))
        if kind == "until":
            st["res"] = torch.zeros(S + 3, **i32)
        else:
            st["cnt"] = torch.zeros((c["mcs"] + 1) * (S + 1), **i32)
    return st


def run(state):
    c, kind = state["case"], state["kind"]
    if kind == "step":
        escg.step_mcs(state["p"], state["lat"], state["t"], c["mcs"],
                      state["cnt"])
        state["t"] += c["mcs"]
        return {"lattice": state["lat"], "counts": state["cnt"]}
    if kind == "sim":
        escg.init(state["p"], state["lat"])
        escg.step_mcs(state["p"], state["lat"], 0, c["mcs"], state["cnt"])
        return {"lattice": state["lat"], "counts": state["cnt"]}
    if kind == "until":
        escg.init(state["p"], state["lat"])
        escg.run_until_extinction(state["p"], state["lat"], 0, c["mcs"],
                                  escg.STOP_FIRST_EXTINCTION, state["res"])
        return {"lattice": state["lat"], "result": state["res"]}
    if kind == "batch":
        escg.batch_run(state["params"], state["offsets"], state["lat"],
                       state["max_mcs"], escg.STOP_FIRST_EXTINCTION, True,
                       state["res"])
        return {"lattices": state["lat"], "results": state["res"]}
    n = c["n"]
    escg.step_batch(state["params"], state["lats"], [state["t"]] * n,
                    state["n_mcs"])
    state["t"] += c["mcs"]
    return {"lattices": state["lats"]}


def work(case):
    """Bytes: every lattice read once and written once (only written where
    the pass initialises it), counts and results written.  flops: integer
    operations, 15 per site-update (a quarter of a Philox4x32-7 call, two
    action tests, the pair's choice and the rule)."""
    c, kind = case, case["kind"]
    if kind == "multi":
        tab = _multi_table(c)
        sites = sum(L * L for L, _, _ in tab)
        return {"bytes": 2.0 * sites,
                "flops": 15.0 * sum(L * L * n for L, _, n in tab)}
    if kind == "batch":
        # the MCS until extinction are not known beforehand: one is certain
        sites = float((_batch_table(c).L.astype(np.int64) ** 2).sum())
        return {"bytes": sites + 4.0 * escg.BATCH_RESULT_WORDS * c["n"],
                "flops": 15.0 * sites}
    sites, row = float(c["L"]) ** 2, 4.0 * (c["S"] + 1)
    if kind == "until":
        return {"bytes": sites + row + 8, "flops": 15.0 * sites}
    return {"bytes": (2.0 if kind == "step" else 1.0) * sites
            + row * (c["mcs"] + 1), "flops": 15.0 * sites * c["mcs"]}


# ---------------------------------------------------------------------------
# The same in numpy, from the definition of the block schedule
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-7 of counters with varying word c0: four uint64 arrays."""
    m = np.uint64(0xFFFFFFFF)
    c0 = np.asarray(c0, np.uint64)
    c1, c2, c3 = (np.full_like(c0, v) for v in (c1, c2, c3))
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(7):
        a, b = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        c0, c1, c2, c3 = ((b >> np.uint64(32)) ^ c1 ^ np.uint64(k0), b & m,
                          (a >> np.uint64(32)) ^ c3 ^ np.uint64(k1), a & m)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _pass(g, t, p, off, c, dom, ab, T1, T2, seed):
    L, Lb = c["L"], c["L"] // 2
    Q = (Lb + 3) // 4
    ox, oy = off & 1, (off >> 1) & 1
    w = np.stack(_philox(np.arange(Lb * Q), t, (3 << 8) | p, 0, seed), 1)
    w = w.reshape(Lb, 4 * Q)[:, :Lb].astype(np.int64)
    s = np.roll(g, (-oy, -ox), (0, 1)).reshape(Lb, 2, Lb, 2)
    s = s.transpose(0, 2, 1, 3).reshape(Lb, Lb, 4).copy()  # A, B, C, D
    first = np.array([0, 2, 0, 1, 0, 1, 0, 1])
    second = np.array([1, 3, 2, 3, 3, 2, 3, 2])
    e = (w >> 3) & (7 if c["moore"] else 3)
    flip = ((w >> (6 if c["moore"] else 5)) & 1).astype(bool)
    ix = np.where(flip, second[e], first[e])[..., None]
    iy = np.where(flip, first[e], second[e])[..., None]
    x = np.take_along_axis(s, ix, 2)[..., 0].astype(np.int64)
    y = np.take_along_axis(s, iy, 2)[..., 0].astype(np.int64)
    u = w >> 8
    ex, sel = u < T1, (u >= T1) & (u < T2)
    rep = ~ex & ~sel
    fight = sel & (x != y) & (x > 0) & (y > 0)
    if ab is not None:
        win = u - T1 < ab[0][x, y]
        lose = ~win & (u - T1 < ab[1][x, y])
    else:
        win, lose = dom[x, y], ~dom[x, y] & dom[y, x]
    nx = np.where(ex, y, np.where(fight & lose, 0,
                                  np.where(rep & (x == 0), y, x)))
    ny = np.where(ex, x, np.where(fight & win, 0,
                                  np.where(rep & (y == 0), x, y)))
    np.put_along_axis(s, ix, nx[..., None].astype(np.uint8), 2)
    np.put_along_axis(s, iy, ny[..., None].astype(np.uint8), 2)
    s = s.reshape(Lb, Lb, 2, 2).transpose(0, 2, 1, 3).reshape(L, L)
    return np.roll(s, (oy, ox), (0, 1))


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind not in ("step", "sim") or c["L"] ** 2 * c["mcs"] > 1.5e7:
        return None
    L, S, seed = c["L"], c["S"], int(seed)
    ex = c["M"] * L * L / 2.0
    tot = (ex + 1.0) + 1.0
    T1 = math.floor(math.ldexp(ex / tot, 24))
    T2 = math.floor(math.ldexp((ex + 1.0) / tot, 24))
    dom = np.zeros((S + 1, S + 1), bool)
    for a in range(S):
        for k in _dominance(S):
            if k % S:
                dom[a + 1, (a + k) % S + 1] = True
    ab = None
    if c["prob"]:
        P = np.zeros((S + 1, S + 1))
        P[1:, 1:] = _probabilities(S)
        P = np.where(dom, P, 0.0)
        A = np.floor(P * (T2 - T1))
        ab = A, A + np.floor(P.T * ((T2 - T1) - A))
    if kind == "sim":
        w = np.stack(_philox(np.arange((L * L + 3) // 4), 0, 1 << 8, 0, seed),
                     1).reshape(-1)[:L * L]
        g = (w * np.uint64(S + 1) >> np.uint64(32)).astype(np.uint8)
    else:
        g = _lattice(L, S, seed).cpu().numpy()
    g = g.reshape(L, L)
    rows = [np.bincount(g.reshape(-1), minlength=S + 1)]
    for t in range(c["mcs"]):
        off = _philox(np.zeros(1), t, 2 << 8, 0, seed)
        for p in range(4):
            g = _pass(g, t, p, int(off[p][0]), c, dom, ab, T1, T2, seed)
        rows.append(np.bincount(g.reshape(-1), minlength=S + 1))
    return {"lattice": g.reshape(-1),
            "counts": np.concatenate(rows).astype(np.int32)}
