"""Runs host code of libescg.so on the CPU with tests/emu/fake_hip.cpp in the
place of the HIP runtime: no kernel runs, the launches are recorded."""
import ctypes as C
import os
import subprocess
import sys
import types

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "emu", "fake_hip.cpp")


def build(out_dir):
    from paper_2508_16639_amd.build import hipcc
    so = os.path.join(out_dir, "fake_hip.so")
    subprocess.check_call([hipcc(), "-shared", "-fPIC", "-O1", "-std=c++17",
                           "--offload-host-only", SRC, "-o", so])
    return so


def run(so, script, *args):
    """Runs `script` (a test file with a main that takes scenario arguments)
    in a process of its own, whose HIP calls go to the fake runtime."""
    r = subprocess.run([sys.executable, script, so, *map(str, args)],
                       cwd=ROOT, capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, PYTHONPATH=ROOT))
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    return r.stdout


class Fake:
    """The library over the fake runtime, in such a process."""

    def __init__(self, so):
        self.dll = C.CDLL(so, mode=C.RTLD_GLOBAL)
        self.dll.fake_launch.restype = C.c_char_p
        self.dll.fake_allocated.restype = C.c_uint64
        # the binding imports torch only to share its HIP runtime
        sys.modules["torch"] = types.ModuleType("torch")
        from paper_2508_16639_amd import escg
        self.escg, self.lib = escg, escg.lib()

    def reset(self, refuse=0xFFFFFFFF, capture=False, words=0,
              stop=0xFFFFFFFF):
        """refuse: the first cooperative launch that fails; words, stop: count
        rows read back have that many words, species die out at row stop."""
        self.dll.fake_reset(refuse, int(capture), words, stop)

    def launches(self):
        out, v = [], (C.c_uint32 * 4)()
        for i in range(self.dll.fake_launches()):
            name = self.dll.fake_launch(i, v).decode()
            out.append(types.SimpleNamespace(
                name=name, cooperative=bool(v[0]), grid=v[1], block=v[2],
                lds=v[3]))
        return out

    def names(self, part):
        return [x for x in self.launches() if part in x.name]

    def params(self, L, S=3, **kw):
        return self.escg.Params(L=L, S=S, dom=self.escg.circulant_dom(S, [1]),
                                ex=1.0, **kw)

    def step(self, p, n, counts=True, static=False):
        lat = np.zeros(p.L * p.L, np.uint8)
        cnt = np.zeros((n + 1) * (p.S + 1), np.uint32)
        fn = (self.lib.escg_step_mcs_static if static
              else self.lib.escg_step_mcs)
        return fn(C.byref(p.c()), lat.ctypes.data, 0, n,
                  cnt.ctypes.data if counts else None, None)

    def until(self, p, n, mode=0):
        lat = np.zeros(p.L * p.L, np.uint8)
        res = np.zeros(p.S + 3, np.uint32)
        return self.lib.escg_run_until_extinction(
            C.byref(p.c()), lat.ctypes.data, 0, n, mode, res.ctypes.data, None)

    def batch(self, ps, ns, mode=0):
        n = len(ps)
        offs = np.cumsum([0] + [p.L * p.L for p in ps]).astype(np.uint64)
        buf = np.zeros(int(offs[-1]), np.uint8)
        res = np.zeros(n * self.escg.BATCH_RESULT_WORDS, np.uint32)
        cps = (self.escg.CParams * n)(*[p.c() for p in ps])
        return self.lib.escg_batch_run(
            n, cps, offs.ctypes.data_as(C.POINTER(C.c_uint64)),
            buf.ctypes.data, None, (C.c_uint32 * n)(*ns), mode, 1,
            res.ctypes.data, None)

    def step_batch(self, ps, ns):
        n = len(ps)
        lats = [np.zeros(p.L * p.L, np.uint8) for p in ps]
        cps = (self.escg.CParams * n)(*[p.c() for p in ps])
        ptr = (C.c_void_p * n)(*[x.ctypes.data for x in lats])
        return self.lib.escg_step_batch(n, cps, ptr, (C.c_uint32 * n)(),
                                        (C.c_uint32 * n)(*ns), None)
