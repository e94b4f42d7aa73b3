"""Coupled blocks whose advanced range (the interior, and one cell more on every side for
the fluxes) ends at, just before and just after a tile or z chunk, in a workspace full of
not-a-numbers: bit for bit the same grid in one piece, whatever the ghost width.
"""
import numpy as np
import pytest

from paper_2608_14048_amd import inputs as I

pytestmark = pytest.mark.gpu

SCHEMES = {"plm": dict(recon="plm", riemann="hlle", integ="rk2"), "ppm": dict(recon="ppm", riemann="hlld", integ="vl2"),
           "dc": dict(recon="dc", riemann="hlld", integ="euler1")}
BLOCKS = [((28, 30, 46), (14, 15, 23), None), ((32, 17, 25), (16, 17, 25), None), ((60, 62, 22), (30, 31, 22), 6),
          ((62, 16, 65), (62, 8, 65), None), ((10, 9, 144), (5, 9, 48), 5)]


@pytest.mark.parametrize("scheme", list(SCHEMES))
@pytest.mark.parametrize("shape,block,ghost", BLOCKS)
def test_coupled_ranges(shape, block, ghost, scheme):
    import torch

    from paper_2608_14048_amd import Domain, Sim

    st, L = I.turbulence_block(shape, seed=4)
    sim = Sim(shape, L, scheme=SCHEMES[scheme])
    torch.cuda.empty_cache()
    poison = torch.full((1 << 24,), float("nan"), dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    del poison
    dom = Domain(shape, block, L, ghost=ghost, scheme=SCHEMES[scheme])
    try:
        sim.set_state(st)
        dom.set_state(st)
        for _ in range(3):
            dt = sim.dt_cfl()
            assert dom.dt_cfl() == dt
            sim.step(dt)
            dom.step()
            assert np.array_equal(dom.state(), sim.state())
    finally:
        dom.close()
        sim.close()
