"""Sphere-box coordinates of the box kernels, run on the host: whatever origin a
diverging sphere leaves, every box node the kernels address lies inside the
lattice (tests/box_node_driver.cpp).  CPU only."""
import os
import subprocess

from paper_1909_01092_amd import build as b


def test_box_nodes_lie_in_the_lattice(tmp_path):
    exe = tmp_path / "box_node"
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "box_node_driver.cpp")
    subprocess.run([b.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I" + b.CSRC,
                    "-I" + os.path.join(b.ROOT, "include"), src, "-o", str(exe)], check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
