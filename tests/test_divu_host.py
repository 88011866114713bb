"""The launch-time division of the HIP path (csrc/divu.h), built for the host
with g++: exact over the whole range of numerators at small divisors, around
every power of two and at random ones, and at each multiple's two sides."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_division_by_a_launch_constant_is_exact(tmp_path):
    exe = str(tmp_path / "divu_driver")
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(HERE, "host", "divu_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 3_000_000
