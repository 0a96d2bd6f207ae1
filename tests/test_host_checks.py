"""Host code of the library where no device memory is to be had: host_checks.cpp,
compiled against libmapmaker.so and its internal header, one check per test."""
import os
import subprocess

import pytest

from paper_1801_08937_amd import build, mapmaker as mm

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_checks(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_checks")
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    lib = os.path.dirname(mm.LIB_PATH)
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC, "-I",
                        build.INCLUDE, "-I", f"{rocm}/include",
                        os.path.join(HERE, "host_checks.cpp"), "-o", exe, mm.LIB_PATH,
                        f"-L{rocm}/lib", "-lamdhip64", f"-Wl,-rpath,{rocm}/lib",
                        f"-Wl,-rpath,{lib}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("check", ["regrid", "p_launch", "tile_keys", "reduction_blocks",
                                   "fft_block", "release", "scratch_sizes",
                                   "pt_forms", "slices"])
def test_host_check(host_checks, check):
    r = subprocess.run([host_checks, check], capture_output=True, text=True, timeout=60)
    if r.returncode == 77:
        pytest.skip("for a machine without a GPU")
    assert r.returncode == 0, r.stdout + r.stderr
