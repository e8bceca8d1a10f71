"""The workspace cache of the digit sorts: what it keeps, lends and gives
back, with a counting allocator (no GPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_workspace_cache_policy(tmp_path):
    exe = str(tmp_path / "workspace_cache")
    subprocess.run(["g++", "-std=c++20", "-O1", "-fsanitize=address,undefined",
                    "-o", exe, os.path.join(HERE, "workspace_cache_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
