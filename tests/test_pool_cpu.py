"""The device-memory pool against a stand-in allocator, on the CPU (pool_check.cpp): fits, bounds, eviction,
the empty-and-retry path, trimming and threads."""
import os
import subprocess

from paper_2606_26297_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_pool_on_a_counted_allocator(tmp_path):
    exe = str(tmp_path / "pool_check")
    subprocess.run([B.CXX, "-std=c++17", "-O1", "-g", "-pthread", *B.HOST, os.path.join(B.CSRC, "qq_pool.cpp"),
                    os.path.join(HERE, "pool_check.cpp"), "-o", exe], check=True, timeout=300)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "pool ok", out.stdout + out.stderr
