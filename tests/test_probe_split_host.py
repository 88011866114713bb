"""The probe's split of a unit's tokens over workgroups (csrc/probe_split.h),
built for the host with g++: whole steps, at most 1024 tokens a workgroup (what
is summed in fp32), within the partials of the workspace, every token once."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_split_keeps_its_bounds(tmp_path):
    exe = str(tmp_path / "probe_split_driver")
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(HERE, "host", "probe_split_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 400_000
