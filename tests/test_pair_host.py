"""The host side of the binned candidate pairs (csrc/pairs.cpp) on the CPU under
AddressSanitizer and UBSan, with launches that are only counted and scripted
read-backs (tests/sanitize/pairs_checks.cpp)."""
import os
import shutil

import pytest

from test_sanitizers import ROOT, build_and_run


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the ROCm headers")
def test_pair_host(tmp_path):
    csrc = os.path.join(ROOT, "paper_2403_09010_amd", "csrc")
    build_and_run(tmp_path, "pairs_checks",
                  [os.path.join(csrc, "pairs.cpp"),
                   os.path.join(ROOT, "tests", "sanitize", "pairs_checks.cpp")],
                  ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                   "-I" + os.path.join(ROOT, "include"), "-I" + csrc])


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_partition_plans(tmp_path):
    """Every plan of a partition fits the kernels that take it."""
    build_and_run(tmp_path, "plan_checks",
                  [os.path.join(ROOT, "tests", "sanitize", "plan_checks.cpp")],
                  ["-I" + os.path.join(ROOT, "paper_2403_09010_amd", "csrc")])


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_device_set_offsets(tmp_path):
    """No offsets of a device set have the packing kernel read outside its codes."""
    build_and_run(tmp_path, "set_checks",
                  [os.path.join(ROOT, "tests", "sanitize", "set_checks.cpp")],
                  ["-I" + os.path.join(ROOT, "paper_2403_09010_amd", "csrc")])


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the ROCm headers")
def test_index_pool(tmp_path):
    """Blocks of freed indexes: what is kept, and who gets it back."""
    csrc = os.path.join(ROOT, "paper_2403_09010_amd", "csrc")
    build_and_run(tmp_path, "pool_checks",
                  [os.path.join(csrc, "index_pool.cpp"),
                   os.path.join(ROOT, "tests", "sanitize", "pool_checks.cpp")],
                  ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                   "-I" + os.path.join(ROOT, "include"), "-I" + csrc])
