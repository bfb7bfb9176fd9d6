"""The observables' column sums at chunk edges (fewer planes than a chunk, one
plane over, several chunks), on walls and periodic axes, against the same sums of
the per-node fields, which another kernel forms.

Bar 1e-11: both are FP64; the gradients add their 18 terms in another order, an
error of about 1e-16 of the densities, and the velocities (kT = 1e-5) are 1e-3.
"""
import numpy as np
import pytest

from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,walls,radius", [
    ((2, 3, 2), 3, 0.0), ((9, 5, 3), 3, 0.0), ((17, 16, 5), 7, 0.0), ((20, 14, 7), 1, 0.0), ((16, 17, 8), 4, 0.0),
    ((14, 15, 18), 6, 3.2), ((70, 40, 33), 0, 4.1), ((30, 12, 130), 3, 2.4)])
def test_columns_against_fields(size, walls, radius):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx, ny, nz = size
    p = workloads.full(dict(nx=nx, ny=ny, nz=nz, walls=walls, init_amp=1e-3, G=1.5, kT=1e-5, g=(1e-5, 2e-5, 5e-5), seed=4,
                            radius=radius))
    sim = Simulation([p, dict(p, seed=5)], "fp64")
    sim.step(3)
    for rep in (0, 1):
        o = sim.observables(rep, profile=True)
        rho, u = sim.fields(rep)
        fluid = rho.sum(axis=0) != 0.0
        cnt = fluid.sum(axis=0)
        uz = np.where(fluid, u[2], 0.0).sum(axis=0) / np.maximum(cnt, 1)
        u2 = float((u * u).sum() / fluid.sum())
        prof = np.asarray(o["uz_profile"]).reshape(uz.shape)
        assert np.abs(prof - uz).max() <= 1e-11 * np.abs(u).max(), (size, rep)
        assert abs(o["u2_mean"] - u2) <= 1e-11 * u2
        assert np.allclose(o["mass"], rho.sum(axis=(1, 2, 3)), rtol=1e-11, atol=0)
    sim.close()
