"""The dust fluid passes that take a workgroup's block of four rows (FP64 donor cell on
grids large enough) and those of single rows that solve both x faces of a cell (small
grids): at the edges of their tiles and chunks against the oracle, and bit for bit against
the other forms on a pattern repeated until those are taken.  Tolerance: the method's FP64
contract, 1e-12 of a class's scale after one step."""
import numpy as np
import pytest

import oracle
from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_parity import STEP_TOL, Pair, assert_close

pytestmark = pytest.mark.gpu


# 16 species: more than 12288 waves of two rows; remainders along every axis, single rows,
# chunks of 8 planes and of more
@pytest.mark.parametrize("shape", [(65, 62, 60), (64, 53, 107), (3, 130, 47), (1, 1500, 5), (70, 1, 1600)])
def test_donor_blocks(shape):
    st, ts = I.dust_drift(shape=shape, nd=16, seed=7, noise=0.3)
    st = np.ascontiguousarray(st, dtype=np.float64).reshape(-1)
    st[4 * int(np.prod(shape)) + 2] = 0.0  # a dust cell below its floor
    pr = Pair(shape, eos="isothermal_hydro", riemann="hlle", integ="imex2p", tstop=ts, gacc=(0.05, -0.02, 0.01),
              recon="dc")
    try:
        dt = oracle.dt_cfl(pr.cfg, st)
        ref = oracle.step(pr.cfg, st, dt)
        pr.sim.set_state(st)
        pr.sim.step(dt)
        assert_close(pr, pr.sim.state(), ref, STEP_TOL, f"donor blocks {shape}")
    finally:
        pr.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("recon,shape,times", [("dc", (70, 13, 22), 13), ("plm", (70, 13, 6), 9),
                                               ("plm", (63, 1, 1), 100), ("dc", (130, 2, 3), 20)])
def test_dust_forms_give_the_same_bits(recon, shape, times, prec):
    """A periodic pattern alone and repeated along y, three steps."""
    nx, ny, nz = shape
    nd = 16
    st, ts = I.dust_drift(shape=shape, nd=nd, seed=8, noise=0.2)
    u = np.asarray(st, dtype=np.float64).reshape(4 * (nd + 1), nz, ny, nx)
    big = np.ascontiguousarray(np.tile(u, (1, 1, times, 1)))
    kw = dict(physics=dict(eos="isothermal_hydro", tstop=tuple(ts), gacc=(0.05, 0.0, 0.0)),
              scheme=dict(recon=recon, riemann="hlle", integ="imex2p", prec=prec))
    a = B.Sim(shape, (1.0, 1.0, 1.0), **kw)
    b = B.Sim((nx, ny * times, nz), (1.0, float(times), 1.0), **kw)
    try:
        a.set_state(u.reshape(-1))
        b.set_state(big.reshape(-1))
        dt = a.dt_cfl()
        for _ in range(3):
            a.step(dt)
            b.step(dt)
        one = a.state().reshape(u.shape)
        assert np.array_equal(b.state().reshape(big.shape), np.tile(one, (1, 1, times, 1)))
    finally:
        a.close()
        b.close()
