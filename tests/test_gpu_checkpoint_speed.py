"""A checkpoint or restore takes about what a copy of its bytes takes: 1.0 to 1.3
times, with 1.5 as the bar (1.9 when every load waited for the store before it)."""
import time

import pytest

from paper_1909_01092_amd import workloads

pytestmark = pytest.mark.gpu


def test_checkpoint_costs_about_a_copy():
    import torch
    from paper_1909_01092_amd.sim import Simulation
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sim = Simulation(workloads.full(dict(nx=130, ny=130, nz=260, walls=3, init_amp=1e-3, G=1.5, kT=1e-5, seed=3)), "fp16")
    sim.step(2)
    ck = sim.checkpoint()
    to = torch.empty_like(ck)

    def best(f):
        t = []
        for _ in range(25):
            torch.cuda.synchronize()
            at = time.perf_counter()
            f()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - at)
        return min(t)

    copy, save, load = best(lambda: to.copy_(ck)), best(sim.checkpoint), best(lambda: sim.restore(ck))
    print(f"copy {copy * 1e6:.0f} us, checkpoint {save * 1e6:.0f}, restore {load * 1e6:.0f}", flush=True)
    assert save < 1.5 * copy and load < 1.5 * copy
    sim.close()
