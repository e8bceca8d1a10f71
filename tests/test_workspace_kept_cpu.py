"""The workspace cache's answer to calls that an allocation of their own would
make slower than the network (no GPU)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_only_kept_workspaces(tmp_path):
    exe = str(tmp_path / "workspace_kept")
    subprocess.run(["g++", "-std=c++20", "-O1", "-fsanitize=address,undefined",
                    "-o", exe, os.path.join(HERE, "workspace_kept_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_no_exception_without_host_memory(tmp_path):
    exe = str(tmp_path / "workspace_noexcept")
    subprocess.run(["g++", "-std=c++20", "-O1",
                    "-o", exe, os.path.join(HERE, "workspace_noexcept_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


def test_idle_streams_make_room(tmp_path):
    exe = str(tmp_path / "workspace_evict")
    subprocess.run(["g++", "-std=c++20", "-O1", "-fsanitize=address,undefined",
                    "-o", exe, os.path.join(HERE, "workspace_evict_driver.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
