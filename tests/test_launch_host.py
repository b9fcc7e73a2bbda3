"""Host test of the kernels' launch arithmetic (csrc/ss_launch.hpp, HIP-free),
compiled with g++: calls of up to 2^31 - 1 rays are launched whole, below HIP's
2^32 threads per launch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_cover_a_call_and_stay_below_the_limit(tmp_path):
    exe = tmp_path / "launch_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "paper_2511_11078_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "launch_test.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all checks passed" in r.stdout
