"""The 8-byte sorts' tile: the library's choice by the number of elements until
a caller sets one, and then the caller's."""
import subprocess
import sys

CHECK = """
from paper_1506_01446_amd import binding as B

def tile(n):
    return B.bitonic_plan_shapes(n, "keys64")[0]["q"]

assert [tile(2**k) for k in (12, 13, 16, 17, 20)] == [12, 11, 11, 13, 13]
assert B.bitonic_get_tuning_value("wide_tile_log2") == 13
for t in (13, 12, 11):
    B.bitonic_set_tuning_value("wide_tile_log2", t)
    assert B.bitonic_get_tuning_value("wide_tile_log2") == t
    assert [tile(2**k) for k in (13, 16, 17, 20)] == [t] * 4, t
print("ok")
"""


def test_a_set_tile_wins():
    r = subprocess.run([sys.executable, "-c", CHECK], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
