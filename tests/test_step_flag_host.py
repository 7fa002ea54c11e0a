"""Slots of COCG's step counts (csrc/step_flag.hpp) in a host program with stand-ins for the runtime:
early returns give their slot back, the copy is taken where none is free or there is no pinned memory,
and threads never share one."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    rocm = "/opt/rocm/include"
    if not shutil.which("g++") or not os.path.isdir(os.path.join(rocm, "hip")):
        pytest.skip("no host compiler or HIP headers")
    exe = str(tmp_path_factory.mktemp("flag") / "step_flag_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}",
                    "-I" + os.path.join(ROOT, "paper_2410_03060_amd", "csrc"), os.path.join(HERE, "step_flag_host.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("args", [[], ["no-pinned-memory"]])
def test_slots(program, args):
    out = subprocess.run([program, *args], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
