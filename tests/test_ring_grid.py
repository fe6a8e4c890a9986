"""The grid of the short-K ring kernel, on the host: no XCD is given more workgroups than its CUs hold at a time."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_walkers_are_balanced_over_the_xcds(tmp_path):
    exe = str(tmp_path / "ring_grid")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-o", exe, os.path.join(HERE, "sanitize", "ring_grid_driver.cpp")])
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
