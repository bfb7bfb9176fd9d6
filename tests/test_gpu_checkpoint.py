"""The form of a checkpoint: populations as one array per component and
direction over the lattice padded by one layer per side, deviations from
w_i rho0_l, population i of node x at padded position x - c_i, zero where no
node pulls from; checked against the exported populations on small lattices of
every wall mask, odd sizes and two replicas, and read back into a context
whose memory was poisoned.

Tolerance: f = w_i (rho0_l + delta_l) + d in FP64 takes three roundings of
numbers below 0.4, each at most 2^-53 relative: 1e-15 holds.
"""
import numpy as np
import pytest

from oracle import oracle as om
from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walls", range(8))
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_checkpoint_form_and_round_trip(walls, prec):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    _, w, _, c = om.basis()
    reps = [workloads.full(dict(nx=13, ny=12, nz=15, walls=walls, init_amp=1e-3, G=1.5, kT=1e-4, radius=2.6,
                                wet_drho=0.1, g=(0.0, 0.0, 1e-4), U0=(0.02, -0.03, 0.04), seed=31)),
            workloads.full(dict(nx=2, ny=5, nz=3, walls=walls, init_amp=1e-3, kT=1e-4, seed=32, replica=1))]
    a = Simulation(reps, prec, fill=0xFF)
    a.step(7)
    ck = a.checkpoint()
    es = 8 if prec == "fp64" else 4
    raw, at = ck.cpu().numpy(), 0
    for r, p in enumerate(reps):
        nx, ny, nz = p["nx"], p["ny"], p["nz"]
        n = 38 * (nx + 2) * (ny + 2) * (nz + 2)
        blk = raw[at:at + n * es].view(np.float64 if es == 8 else np.float32).astype(np.float64)
        at += n * es
        blk = blk.reshape(2, 19, nz + 2, ny + 2, nx + 2)
        f, st = a.populations(r), a.particle_state(r)
        fluid = f[0, 0] != 0
        seen = np.zeros(blk.shape, bool)
        for i in range(19):
            z, y, x = 1 - c[i][2], 1 - c[i][1], 1 - c[i][0]
            at_i = (slice(None), i, slice(z, z + nz), slice(y, y + ny), slice(x, x + nx))
            seen[at_i] = True
            for l in range(2):
                got = w[i] * (p["rho0"][l] + st["delta"][l]) + blk[at_i][l]
                assert np.abs(got - f[l, i])[fluid].max() < 1e-15, (walls, prec, r, i, l)
        assert not blk[~seen].any()
    b = Simulation(reps, prec, fill=0xFF)
    b.restore(ck)
    a.step(9)
    b.step(9)
    for r in range(len(reps)):
        assert np.array_equal(a.populations(r), b.populations(r))
        assert np.array_equal(a.particle_state(r)["X"], b.particle_state(r)["X"])
    a.close()
    b.close()
