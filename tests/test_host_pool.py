"""The pool that a handle's device memory comes from (csrc/host_copy.hip) without a GPU: built
for the host with stand-ins for the HIP calls (tests/c/host_pool.cpp), on a device of a few
megabytes.  Memory that one of a handle's two pools holds without use serves the other
before an allocation fails; blocks never overlap; everything goes back."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = "/opt/rocm/include"


def test_pools_share_the_device(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "host_pool")
    subprocess.run([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{HIP_INCLUDE}",
                    f"-I{os.path.join(ROOT, 'include')}",
                    f"-I{os.path.join(ROOT, 'paper_1511_02433_amd', 'csrc')}",
                    os.path.join(ROOT, "tests", "c", "host_pool.cpp"), "-pthread", "-o", exe],
                   check=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
