"""Parts of the kernels' sources that are plain C++, compiled for the CPU: the programs under tests/host check them over ranges
that no GPU test could cover, and print "ok"."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("name", ["chunk_groups", "edge_bounds", "list_rules", "threshold_search"])
def test_host_unit(tmp_path, name):
    exe = str(tmp_path / name)
    # (signed overflow ends the program instead of wrapping)
    cmd = ["g++", "-std=c++17", "-O2", "-fsanitize=signed-integer-overflow", "-fsanitize-undefined-trap-on-error",
           "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2508_15706_amd", "csrc"), os.path.join(HERE, "host", name + ".cpp"), "-o", exe]
    subprocess.run(cmd, check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert (r.returncode, r.stdout.strip()) == (0, "ok"), r.stdout + r.stderr
