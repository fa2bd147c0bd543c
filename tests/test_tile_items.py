"""The order in which the tile GEMM hands its work items to workgroups, driven on the host by a small C++ program
(tests/host/tile_items_driver.cpp) that includes the kernel's own header."""
import os
import subprocess

from paper_2306_15799_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_item_once_and_no_id_without_a_tile(tmp_path):
    exe = str(tmp_path / "tile_items")
    subprocess.run([build.find_hipcc(), "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-I",
                    os.path.join(build.ROOT, "include"), "-I", build.CSRC, os.path.join(HERE, "host", "tile_items_driver.cpp"),
                    "-o", exe], check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert "all expectations held" in res.stdout
