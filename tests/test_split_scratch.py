"""The host side of products that the library cuts by itself (which stream may use which part of the scratch space, what is refused, what
each of two launches is given), without a GPU: split_scratch_host.cpp runs it on a stand-in for the HIP runtime."""
import os
import subprocess

import pytest

from paper_2506_06472_amd import binding, build

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    binding.lib()
    out = str(tmp_path_factory.mktemp("split_scratch") / "host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
                    os.path.join(HERE, "split_scratch_host.cpp"), build.LIB, "-o", out, f"-Wl,-rpath,{os.path.dirname(build.LIB)}",
                    "-rdynamic", "-Wl,--unresolved-symbols=ignore-in-shared-libs"], check=True)
    return out


@pytest.mark.parametrize("name", ["cuts_and_waits", "refuses_accumulate_with_residual", "a_failed_record_ends_the_sharing",
                                  "leaves_streams_of_other_devices_alone", "large_products_of_four_streams_do_not_wait",
                                  "large_products_share_no_bytes_with_a_running_one", "streams_outputs_by_the_size_of_the_product",
                                  "a_second_launch_goes_on_where_the_first_ends"])
def test_split_scratch(program, name):
    r = subprocess.run([program, name], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
