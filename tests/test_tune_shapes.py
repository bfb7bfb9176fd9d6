"""The tuner's candidate shapes hold the one the context starts with
(tests/tune_shapes_driver.cpp).  CPU only."""
import os
import subprocess

from paper_1909_01092_amd import build as b


def test_tuner_times_the_shape_a_context_has(tmp_path):
    exe = tmp_path / "tune_shapes"
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tune_shapes_driver.cpp")
    subprocess.run([b.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I" + b.CSRC,
                    "-I" + os.path.join(b.ROOT, "include"), src, "-o", str(exe)], check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
