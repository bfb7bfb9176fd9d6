"""Rounding of the general relaxation is written down and not left to the
compiler: the noise of a mode is fused onto the relaxed mode (host run,
tests/relax_driver.cpp), and FP16 results do not depend on which nodes are a
tile's own and which its neighbours' halo (GPU)."""
import os
import subprocess

import numpy as np
import pytest

from paper_1909_01092_amd import build as b, workloads

MRT = dict(tau_shear=0.8, tau_bulk=1.1, tau_mom=0.9, tau_ghost=1.3)


def test_noise_is_fused_onto_the_relaxed_mode(tmp_path):
    exe = tmp_path / "relax"
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "relax_driver.cpp")
    subprocess.run([b.HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-ffp-contract=off", "-I" + b.CSRC,
                    src, "-o", str(exe)], check=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("kT", [0.0, 1e-5])
def test_fp16_general_relaxation_does_not_depend_on_the_tiles(kT):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = workloads.full(dict(nx=56, ny=56, nz=40, walls=3, init_amp=1e-3, G=1.5, kT=kT, seed=3, g=(0.0, 0.0, 1e-5),
                            radius=4.3, wet_drho=0.1, **MRT))
    got = []
    for block, cz in ((256, 3), (512, 5), (1024, 40)):
        sim = Simulation(p, "fp16")
        sim.set_launch(block, cz)
        sim.step(12)
        got.append(sim.populations())
        sim.close()
    assert np.array_equal(got[0], got[1])
    assert np.array_equal(got[0], got[2])
