"""The PPM limiters where their conditions tie: states drawn from a few values, so that
neighbouring differences are often exactly zero, equal or opposite and parabolas sit
exactly on the bounds of overshoot (along x, y and z, at ragged tiles), FP64 against the
oracle at the method's 1e-12 of a class's scale after one step; and a not-a-number cell
is still reported after a step in both precisions.  The flow is everywhere forward and
supersonic along the three axes, so that no mass flux ties with zero: the upwind choice of
the edge EMFs is discontinuous there, and the sign of a flux of rounding errors decides it.
"""
import numpy as np
import pytest

import oracle
from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_parity import STEP_TOL, Pair, Pair32, assert_close

pytestmark = pytest.mark.gpu


def stepped_state(shape, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nz = shape
    full = (nz, ny, nx)
    pick = lambda *v: rng.choice(np.array(v), size=full)
    pots = [rng.choice(np.array([-1.0, 0.0, 1.0]), size=full) / (8 * max(shape)) for _ in range(3)]
    b = I.faces_from_potential(*pots, 1.0 / nx, 1.0 / ny, 1.0 / nz)
    return I.mhd_state(pick(0.5, 0.75, 1.0, 1.5), pick(3.75, 4.0, 4.25), pick(3.75, 4.0, 4.25),
                       pick(3.75, 4.0, 4.25), pick(0.5, 0.75, 1.0) * 1.5, b[0] + 0.5, b[1] - 0.25, b[2] + 0.25)


@pytest.mark.parametrize("riemann", ["hlld", "hlle"])
@pytest.mark.parametrize("shape", [(16, 16, 8), (33, 18, 7), (5, 3, 4)])
def test_ppm_ties(shape, riemann):
    st = stepped_state(shape, 2)
    pr = Pair(shape, recon="ppm", riemann=riemann, integ="rk2")
    try:
        dt = oracle.dt_cfl(pr.cfg, st)
        ref = oracle.step(pr.cfg, st, dt)
        pr.sim.set_state(st)
        pr.sim.step(dt)
        assert_close(pr, pr.sim.state(), ref, STEP_TOL, f"ppm ties {riemann} {shape}")
    finally:
        pr.close()


@pytest.mark.parametrize("make", [Pair, Pair32])
@pytest.mark.parametrize("field", range(8))
def test_ppm_reports_a_nan_cell(make, field):
    shape = (16, 12, 10)
    st = stepped_state(shape, 3)
    n = int(np.prod(shape))
    pr = make(shape, recon="ppm", riemann="hlld")
    try:
        dt = oracle.dt_cfl(pr.cfg, st)
        st[field * n + n // 2 + 5] = np.nan
        pr.sim.set_state(st)
        with pytest.raises(B.MhdError) as e:
            pr.sim.step(dt)
            pr.sim.dt_cfl()
        assert e.value.code == -5
    finally:
        pr.close()
