"""The adjoint's node kernels at tile edges: ragged last tiles, one-row tiles,
each wall mask (the force's wall-mirror sources come from the staged tile), a
sphere near or across the faces.  FP64 against the oracle's adjoint.

Bars as for the other FP64 adjoint cases: 1e-12 on J, 1e-9 on each gradient
component.
"""
import pytest

from oracle.oracle import OracleSim
from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,walls,X0", [
    ((37, 14, 12), 1, (4.1, 13.6, 0.2)), ((37, 14, 12), 2, (0.3, 6.5, 11.7)), ((20, 13, 15), 4, (19.8, 0.2, 6.9)),
    ((12, 22, 13), 5, (5.6, 21.7, 6.4)), ((12, 15, 14), 6, (0.1, 7.2, 6.6)), ((130, 12, 13), 7, (60.4, 5.4, 6.3)),
    ((129, 12, 12), 0, (128.7, 0.1, 11.8))])
def test_adjoint_tiles(size, walls, X0):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nx, ny, nz = size
    p = workloads.full(dict(nx=nx, ny=ny, nz=nz, walls=walls, init_amp=1e-3, G=1.5, kT=1e-5, seed=12, g=(0.0, 0.0, 5e-5),
                            radius=2.6, rho_p=2.0, wet_drho=0.1, X0=X0, U0=(0.03, -0.02, 0.05), W0=(0.01, 0.0, -0.01)))
    print(size, walls, flush=True)
    Jo, go = OracleSim(p).adjoint(8)
    sim = Simulation(p, "fp64")
    J, grad = sim.adjoint(8, 3)
    assert abs(J - Jo) <= 1e-12 * abs(Jo)
    for k in range(5):
        assert abs(grad[k] - go[k]) <= 1e-9 * abs(go[k]) + 1e-14, (k, grad[k], go[k])
    sim.close()
