"""A sphere that diverges: far lighter than the fluid, shaken by far too much
noise, or driven past several periods of its channel in one step (the external
force alone adds g/2 to its velocity per step).  The run ends in LBM_EUNSTABLE,
and the replicas beside it in the batch keep their bits."""
import numpy as np
import pytest

from paper_1909_01092_amd import _capi, workloads

pytestmark = pytest.mark.gpu
BASE = dict(nx=16, ny=16, nz=24, walls=3, init_amp=1e-3, G=1.5, kT=1e-5, seed=3, radius=2.5, g=(0.0, 0.0, 1e-4),
            wet_drho=0.1)


@pytest.mark.parametrize("prec", ["fp32", "fp64", "fp16"])
@pytest.mark.parametrize("walls,bad", [(3, dict(rho_p=0.02)), (0, dict(rho_p=0.02)), (4, dict(rho_p=0.1)),
                                       (3, dict(kT=0.03)), (3, dict(g=(0.0, 0.0, 150.0))),
                                       (0, dict(g=(-1e5, 3e3, 1e12)))])
def test_runaway_sphere(prec, walls, bad):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(prec, walls, bad, flush=True)
    good = [workloads.full(dict(BASE, walls=walls, replica=r)) for r in range(2)]
    away = workloads.full(dict(BASE, walls=walls, replica=2, **bad))
    both = Simulation([good[0], away, good[1]], prec)
    alone = Simulation(good, prec)
    for s in (both, alone):
        s.set_launch(256, 3)
        s.step(12)
    lost = both.particle_state(1, allow_unstable=True)
    with pytest.raises(_capi.LbmError) as e:
        both.particle_state(1)
    assert e.value.code == _capi.LBM_EUNSTABLE
    if "g" in bad:
        assert not np.abs(lost["U"][2]) < 2 * 24  # several periods in a step
    for k, r in ((0, 0), (2, 1)):
        a, b = both.particle_state(k), alone.particle_state(r)
        for key in ("X", "U", "W", "F"):
            assert np.array_equal(a[key], b[key]), key
        assert np.array_equal(both.populations(k), alone.populations(r))
    both.close()
    alone.close()
