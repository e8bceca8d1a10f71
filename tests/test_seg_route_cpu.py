"""Which segments of a segmented sort go by digits: the rules of segroute.hpp
on the host (no GPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_seg_route(tmp_path):
    exe = str(tmp_path / "seg_route")
    subprocess.run(["g++", "-std=c++20", "-O1", "-fsanitize=address,undefined",
                    "-o", exe, os.path.join(HERE, "seg_route_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
