"""Grids on both sides of the sizes at which a workgroup of the MHD kernels takes one z
plane and not two (768 of them at once; the flux and the CT kernel's lines differ), odd
plane counts and single planes among them: state and time step after two steps bit for bit
those of a one-block batch, whose workgroups take chunks of up to 24 (flux) and 64 planes.
"""
import numpy as np
import pytest

from paper_2608_14048_amd import binding as B
from tests.test_gpu_parity import random_mhd

pytestmark = pytest.mark.gpu

# planes of 16 x 16 and of 64 x 8 tiles: 768 and one more, far below, only one kernel below
SHAPES = [(16, 16, 768), (16, 16, 769), (17, 17, 193), (65, 8, 3), (3, 200, 5), (130, 24, 7), (16, 130, 86), (9, 9, 1)]


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("recon,riemann,integ", [("ppm", "hlld", "vl2"), ("plm", "hlle", "rk2")])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_and_two_plane_workgroups(shape, recon, riemann, integ, prec):
    length = tuple(v / max(shape) for v in shape)
    st = random_mhd(shape, 8, length, amp=0.2)
    scheme = dict(recon=recon, riemann=riemann, integ=integ, prec=prec)
    sim, bt = B.Sim(shape, length, scheme=scheme), B.Batch([shape], [length], scheme=scheme)
    try:
        sim.set_state(st)
        bt.set_state([st])
        for _ in range(2):
            assert sim.dt_cfl() == bt.dt_cfl()[0]
            sim.step(sim.dt_cfl())
            bt.step()
        assert sim.dt_cfl() == bt.dt_cfl()[0]
        assert np.array_equal(sim.state(), bt.state())
    finally:
        sim.close()
        bt.close()
