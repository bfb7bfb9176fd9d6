"""The launch shape a new context starts with: admissible for every lattice
(block holds a row, LDS fits: the first step runs), a z-chunk of one plane on a
tiny lattice, blocks of 512 or 1024 on wide rows, never 1024 threads in the
forms that would spill there, and the same results as another shape (bitwise in
FP32, 1e-14 in FP64, where the compiler rounds the block forms differently).
"""
import numpy as np
import pytest

from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu
MRT = dict(tau_shear=0.8, tau_bulk=1.1, tau_mom=0.9, tau_ghost=1.3)


@pytest.mark.parametrize("size,prec,more", [
    ((2, 3, 2), "fp32", {}), ((16, 16, 32), "fp32", {}), ((24, 24, 48), "fp64", {}), ((33, 20, 40), "fp32", MRT),
    ((192, 40, 16), "fp32", {}), ((150, 64, 64), "fp16", {}), ((256, 30, 12), "fp64", {}), ((250, 64, 40), "fp32", MRT)])
def test_default_shape(size, prec, more):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx, ny, nz = size
    p = workloads.full(dict(nx=nx, ny=ny, nz=nz, walls=3, init_amp=1e-3, G=1.5, kT=1e-5, seed=5, **more))
    a, b = Simulation(p, prec), Simulation(p, prec)
    block, cz = a.get_launch()
    print(size, prec, block, cz, flush=True)
    assert block in (256, 512, 1024) and block >= nx and 1 <= cz <= 32
    assert not (block == 1024 and (prec == "fp64" or more))
    if size in ((16, 16, 32), (24, 24, 48)):
        assert cz == 1
    b.set_launch(256, 3)
    a.step(4)
    b.step(4)
    fa, fb = a.populations(), b.populations()
    if prec == "fp64":
        assert np.abs(fa - fb).max() <= 1e-14 * np.abs(fb).max()
    else:
        assert np.array_equal(fa, fb)
    a.set_launch(block, 0)
    assert a.get_launch() == (block, cz)
    a.close()
    b.close()
