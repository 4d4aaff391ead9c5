"""Host emulation of the patch kernel's and the small-lattice kernel's phases
against the oracle, byte for byte: the device headers compiled for the host
as in test_kernel_emulation_cpu.py, a workgroup's threads one after another
(a pass reads one copy of the lattice and writes another)."""
import os
import subprocess

import pytest

from tests.test_kernel_emulation_cpu import (EMU, emu_dir,  # noqa: F401
                                             pytestmark)


@pytest.mark.parametrize("prog,expect", [("emu_patch", "patch cases ok"),
                                         ("emu_whole", "whole cases ok")])
def test_device_logic_matches_oracle(emu_dir, prog, expect):  # noqa: F811
    exe = os.path.join(emu_dir, prog)
    subprocess.check_call(
        ["g++", "-O1", "-std=c++17", f"-I{EMU}", f"-I{emu_dir}/src",
         os.path.join(EMU, prog + ".cpp"), os.path.join(emu_dir, "orc.o"),
         "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    last = r.stdout.strip().splitlines()[-1]
    assert r.returncode == 0, r.stdout[-2000:]
    n_ok, n = last.split()[0].split("/")
    assert expect in last and n_ok == n and int(n) > 0, last
