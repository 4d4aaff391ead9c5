"""Host emulation of the kernel that keeps two copies of a lattice in LDS
(passes of several quads a thread, the windows between two tests of the stop
condition), as in test_kernel_emulation_cpu.py."""
import os
import subprocess

from tests.test_kernel_emulation_cpu import (EMU, emu_dir,  # noqa: F401
                                             pytestmark)


def test_passes_and_windows(emu_dir):  # noqa: F811
    exe = os.path.join(emu_dir, "emu_pair")
    subprocess.check_call(
        ["g++", "-O1", "-std=c++17", f"-I{EMU}", f"-I{emu_dir}/src",
         os.path.join(EMU, "emu_pair.cpp"), os.path.join(emu_dir, "orc.o"),
         "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    last = r.stdout.strip().splitlines()[-1]
    assert r.returncode == 0, r.stdout[-2000:]
    n_ok, n = last.split()[0].split("/")
    assert "pair cases ok" in last and n_ok == n and int(n) > 4000, last
