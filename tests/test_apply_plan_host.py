"""Host checks of the apply planner (no GPU needed): a C++ program linked
against the library sweeps sizes through plan_apply."""
import os
import subprocess

import pytest

from paper_2607_12969_amd import lrc

HERE = os.path.dirname(os.path.abspath(__file__))


def build_host(tmp_path, source):
    """Compiles tests/<source> against the built library; returns the program."""
    lrc.lib()
    exe = str(tmp_path / source.split(".")[0])
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, source), lrc.LIB_PATH, "-Wl,-rpath," + os.path.dirname(lrc.LIB_PATH),
                    "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64", "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("sweep", ["scratch", "memory", "route"])
def test_plans_fit(tmp_path, sweep):
    """Every FP32 call that the allocation-free entry accepts fits its scratch;
    every call still runs where only the memory of the plan without the split is
    free; and the split runs at the sizes and ranks where it gains."""
    r = subprocess.run([build_host(tmp_path, "apply_plan_host.cpp"), sweep], capture_output=True, text=True, timeout=300)
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_factor_routes(tmp_path):
    """A^T Q straight from memory only at the sizes where that was the faster
    route; the sketch's tiles by the number of test vectors."""
    r = subprocess.run([build_host(tmp_path, "factor_plan_host.cpp")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
