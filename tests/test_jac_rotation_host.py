"""The Jacobi rotation on the host (no GPU needed): both lanes of a pair reach the
same decision and opposite angles from their exchanged norms."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_both_lanes_of_a_pair_agree(tmp_path):
    exe = str(tmp_path / "jac_rotation_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", os.path.join(HERE, "jac_rotation_host.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
