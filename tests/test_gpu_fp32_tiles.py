"""The FP32-bulk flux/update kernels on both sides of the rule that picks 32 x 8 or
16 x 16 tiles, at partial and whole tiles of both: bit for bit against every tile shape
of a one-block batch (the same tile bodies), and within the 2e-6 of one rounded step of
the other FP32 tests against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_parity import FP32_STEP_TOL, Pair32, class_errors

pytestmark = pytest.mark.gpu

# 32 x 8 tiles are no more than 16 x 16 ones for the first six, more for the others
SHAPES = [(32, 8, 9), (31, 33, 6), (17, 16, 8), (33, 7, 12), (64, 41, 5), (96, 24, 16), (16, 16, 8), (40, 16, 6),
          (12, 30, 7)]
SCHEMES = [("ppm", "hlld", "vl2"), ("plm", "hlle", "rk2")]


@pytest.mark.parametrize("recon,riemann,integ", SCHEMES)
@pytest.mark.parametrize("shape", SHAPES)
def test_fp32_tile_shapes_agree(shape, recon, riemann, integ):
    st = I.turbulence_block(shape, seed=3)[0]
    scheme = dict(recon=recon, riemann=riemann, integ=integ, prec="fp32_bulk")
    length = tuple(v / max(shape) for v in shape)
    pr = Pair32(shape, length=length, recon=recon, riemann=riemann, integ=integ)
    bt = B.Batch([shape], [length], scheme=scheme)
    try:
        dt = oracle.dt_cfl(pr.cfg, st)
        ref = oracle.step(pr.cfg, st, dt)
        pr.sim.set_state(st)
        pr.sim.step(dt)
        got = pr.sim.state()
        assert max(class_errors(pr, got, ref).values()) <= FP32_STEP_TOL
        for shp in range(3):
            bt.set_tile_shapes([shp])
            bt.set_state([st])
            bt.step(np.array([dt]))
            assert np.array_equal(bt.state()[bt.block_slices()[0]], got), shp
    finally:
        bt.close()
        pr.close()
