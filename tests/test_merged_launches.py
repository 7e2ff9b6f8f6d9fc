"""Which neighbours of the schedule go out in one launch, without a GPU (merge_host.cpp)."""
import os
import subprocess

import pytest

from paper_2506_06472_amd import binding, build

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    binding.lib()
    out = str(tmp_path_factory.mktemp("merge") / "host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", os.path.join(HERE, "merge_host.cpp"),
                    build.LIB, "-o", out, f"-Wl,-rpath,{os.path.dirname(build.LIB)}", "-Wl,--unresolved-symbols=ignore-in-shared-libs"], check=True)
    return out


def test_updates_of_one_launch_share_no_memory(program):
    r = subprocess.run([program, "independent"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
