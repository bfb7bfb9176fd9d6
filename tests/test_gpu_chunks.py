"""The main kernel over z-chunks of one, two, three and all planes, where its
loads run one plane ahead: tiles whose last rows or lanes hold no node, walls
and periodic axes, a sphere on the faces (solid nodes, wetting densities), 16-
and 32-bit storage and 64-bit, against the oracle.

Bars as in the parity tests: 1e-12 (FP64), 1e-6 and 1e-5 on the deviations
(FP32); FP16 storage: its relative deviations are rounded to 11 bits once per
step, so 2^-11 per step on the deviations.
"""
import pytest

from oracle.oracle import OracleSim
from paper_1909_01092_amd import workloads
from test_gpu_parity import compare

pytestmark = pytest.mark.gpu
STEPS = 6
BARS = {"fp64": (1e-12, 1e-12), "fp32": (1e-6, 1e-5), "fp16": (1e-2, STEPS * 2.0 ** -11)}


@pytest.mark.parametrize("prec", ["fp32", "fp64", "fp16"])
@pytest.mark.parametrize("walls", [0, 4, 7])
def test_chunks_against_oracle(prec, walls):
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = workloads.full(dict(nx=20, ny=15, nz=14, walls=walls, init_amp=1e-3, G=1.5, kT=1e-5, radius=3.1, wet_drho=0.1,
                            X0=(9.7, 7.2, 0.4 if not walls & 4 else 6.3), U0=(0.02, -0.01, 0.03), seed=77))
    ref = OracleSim(p)
    ref.step(STEPS)
    for block, cz in ((256, 1), (256, 2), (512, 3), (256, 14), (512, 14)):
        sim = Simulation(p, prec)
        sim.set_launch(block, cz)
        sim.step(STEPS)
        compare(sim, ref, *BARS[prec], what=f"{prec} walls {walls} {block} x {cz}")
        sim.close()
