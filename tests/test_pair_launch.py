"""CPU check of the launch shapes of the two-step and one-launch two-density
kernels: every site of a grid has one owner for any size, precision and
override (tests/pair_launch_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pair_launch_covers_the_grid(tmp_path):
    exe = tmp_path / "pair_launch_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1412_6238_amd", "csrc"),
                           os.path.join(ROOT, "tests", "pair_launch_check.cpp"), "-o", str(exe)])
    env = {k: v for k, v in os.environ.items() if not k.startswith("LBE_CSF_")}
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.split()[1]) > 500000
