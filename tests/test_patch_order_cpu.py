"""Host emulation of runs on patches that end before their first halo exchange
(as in test_kernel_emulation_cpu.py): no order among the patches is needed
where they read a copy of the lattice."""
import os
import subprocess

from tests.test_kernel_emulation_cpu import (EMU, emu_dir,  # noqa: F401
                                             pytestmark)


def test_patches_one_after_the_other(emu_dir):  # noqa: F811
    exe = os.path.join(emu_dir, "emu_patch_order")
    subprocess.check_call(
        ["g++", "-O1", "-std=c++17", f"-I{EMU}", f"-I{emu_dir}/src",
         os.path.join(EMU, "emu_patch_order.cpp"),
         os.path.join(emu_dir, "orc.o"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    last = r.stdout.strip().splitlines()[-1]
    assert r.returncode == 0, r.stdout[-2000:]
    n_ok, n = last.split()[0].split("/")
    assert "order cases ok" in last and n_ok == n and int(n) > 0, last
