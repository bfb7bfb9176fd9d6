"""Contexts whose populations exceed the cache before memory store them non-
temporally.  Two copies of a lattice in one context (over the limit) against one
alone (under it): the same numbers, bit for bit, in each form that has the branch
(rows of 64 and 32 nodes; walls, whose ghost rows are stored plainly, and periodic
axes; a sphere).
"""
import numpy as np
import pytest

from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu
MRT = dict(tau_shear=0.8, tau_bulk=1.1, tau_mom=0.9, tau_ghost=1.3)


@pytest.mark.parametrize("prec,size,more", [
    ("fp32", (64, 64, 128), dict(walls=3, kT=1e-5)), ("fp32", (32, 48, 400), dict(walls=4, kT=0.0, radius=3.3, wet_drho=0.1)),
    ("fp32", (64, 64, 128), dict(walls=0, kT=1e-5, **MRT)), ("fp64", (32, 40, 220), dict(walls=3, kT=1e-5, radius=3.3)),
    ("fp64", (32, 40, 220), dict(walls=7, kT=1e-5, **MRT))])
def test_streamed_stores(prec, size, more):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx, ny, nz = size
    p = workloads.full(dict(nx=nx, ny=ny, nz=nz, init_amp=1e-3, G=1.5, g=(0.0, 0.0, 1e-5), seed=9, **more))
    mb = nx * (ny + 2) * (nz + 2) * 38 * 2 * (4 if prec == "fp32" else 8) / 1e6
    assert mb < 300 < 2 * mb
    one, two = Simulation(p, prec), Simulation([p, p], prec)
    for s in (one, two):
        s.set_launch(256, 3)
        s.step(4)
    f = one.populations()
    for rep in (0, 1):
        assert np.array_equal(f, two.populations(rep)), (prec, size, rep)
    one.close()
    two.close()
