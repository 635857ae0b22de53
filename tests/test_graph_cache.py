"""The cache of captured iteration chunks (csrc/graph_cache.h), on the host: a solve that pauses
for the explicit Gram has two chunks per precision, and the next equal solve captures none.
"""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_equal_solves_capture_once(tmp_path):
    exe = tmp_path / "graph_cache"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-Wall",
                           os.path.join(HERE, "sanitize", "graph_cache.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
