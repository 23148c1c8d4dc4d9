"""A batch and its members may be destroyed in either order (a garbage collector finalises the objects of a
reference cycle in any): no call on a freed handle's stream, nothing freed twice, nothing left."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_batch_and_members_in_any_order(tmp_path):
    exe = str(tmp_path / "lifetimes")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "lifetime_selftest.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
