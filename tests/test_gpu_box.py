"""The sphere's box kernels at box sizes where their sums split differently:
fewer workgroups than one column pass (edge 12, 27 workgroups), a ragged last
workgroup (edge 16), more than three partials per column (edge 22 and 36: 167
and 729) and more workgroups than one window of the event totals (edge 52:
2197); fast spheres, so that many workgroups have cover and uncover events.
FP64 against the oracle.

Bars as for the other FP64 sphere cases: 1e-12 on populations, counts exact,
1e-10 on the sphere's vectors.
"""
import numpy as np
import pytest

from oracle.oracle import OracleSim
from paper_1909_01092_amd import workloads
from test_gpu_parity import compare, compare_particle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius,n", [(3.0, 14), (4.4, 18), (7.7, 24), (14.6, 38), (22.6, 54)])
def test_box_sizes_against_oracle(radius, n):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = workloads.full(dict(nx=n, ny=n + 1, nz=n + 2, walls=0, init_amp=1e-3, G=1.5, kT=1e-5, radius=radius,
                            wet_drho=0.1, X0=(n - 0.7, n / 2.0, 0.3), U0=(0.11, -0.07, 0.23), W0=(0.004, 0.002, -0.003),
                            seed=41))
    sim, ref = Simulation(p, "fp64"), OracleSim(p)
    sim.step(5)
    ref.step(5)
    compare(sim, ref, 1e-12, what=f"R = {radius}")
    pg, po = compare_particle(sim, ref, 1e-10, what=f"R = {radius}")
    assert po["n_covered"] > 0 and po["n_uncovered"] > 0
    assert pg["n_links"] == po["n_links"] and pg["n_fluid"] == po["n_fluid"]
    assert np.abs(pg["delta"] - po["delta"]).max() <= 1e-10 * np.abs(po["delta"]).max()
    sim.close()
