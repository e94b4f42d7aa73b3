"""The dust fluid passes at the edges of their tiles (64 columns x 1 or 2 rows, a wave
each): partial and whole tiles in x, odd row counts, single rows and planes, grids below
and above the size at which a wave takes two rows.  The noise is strong enough that
every limiter branch occurs.  Tolerances: the method's FP64 contract (1e-12 of a class's
scale after one step) and, FP32, the 2e-6 of one rounded step of the other FP32 tests.
"""
import numpy as np
import pytest

import oracle
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_parity import FP32_DUST_STEP_TOL, STEP_TOL, Pair, PairDust32, assert_close

pytestmark = pytest.mark.gpu

SMALL = [(1, 1, 5), (63, 3, 4), (64, 2, 3), (65, 5, 6), (130, 1, 9), (3, 7, 2)]
TWO_ROWS = [(130, 21, 30), (64, 62, 33)]  # with 16 species: more than 4096 waves of two rows


@pytest.mark.parametrize("recon", ["plm", "dc"])
@pytest.mark.parametrize("nd,shape", [(2, s) for s in SMALL] + [(16, s) for s in TWO_ROWS])
def test_dust_tile_edges(recon, nd, shape):
    st, ts = I.dust_drift(shape=shape, nd=nd, seed=5, noise=0.3)
    kw = dict(tstop=ts, gacc=(0.05, -0.02, 0.01), recon=recon)
    for make, tol in ((lambda: Pair(shape, eos="isothermal_hydro", riemann="hlle", integ="imex2p", **kw), STEP_TOL),
                      (lambda: PairDust32(shape, **kw), FP32_DUST_STEP_TOL)):
        pr = make()
        try:
            dt = oracle.dt_cfl(pr.cfg, st)
            ref = oracle.step(pr.cfg, st, dt)
            pr.sim.set_state(st)
            assert abs(pr.sim.dt_cfl() - dt) <= 1e-14 * dt
            pr.sim.step(dt)
            got = pr.sim.state()
            assert_close(pr, got, ref, tol, f"dust {recon} nd={nd} {shape}")
            after = oracle.dt_cfl(pr.cfg, got)
            assert abs(pr.sim.dt_cfl() - after) <= 1e-13 * after
        finally:
            pr.close()


def test_dust_result_does_not_depend_on_the_tiling():
    """The same periodic pattern on a grid one period wide (one row per wave) and on its
    tiling three times along y (two rows per wave) gives the same bits in every copy."""
    nx, ny, nz, nd = 70, 15, 24, 16
    st, ts = I.dust_drift(shape=(nx, ny, nz), nd=nd, seed=6, noise=0.2)
    u = st.reshape(4 * (nd + 1), nz, ny, nx)
    big = np.ascontiguousarray(np.tile(u, (1, 1, 3, 1))).reshape(-1)
    a = PairDust32((nx, ny, nz), ts)
    b = PairDust32((nx, 3 * ny, nz), ts)
    try:
        # equal spacings: the second box is three times as long in y
        b.sim.close()
        from paper_2608_14048_amd import binding as B
        b.sim = B.Sim((nx, 3 * ny, nz), (1.0, 3.0, 1.0),
                      physics=dict(eos="isothermal_hydro", tstop=tuple(ts), gacc=(0.05, 0.0, 0.0)),
                      scheme=dict(recon="plm", riemann="hlle", integ="imex2p", courant=0.3, prec="fp32_bulk"))
        a.sim.set_state(st)
        b.sim.set_state(big)
        dt = a.sim.dt_cfl()
        assert b.sim.dt_cfl() == dt
        for _ in range(3):
            a.sim.step(dt)
            b.sim.step(dt)
        ga = a.sim.state().reshape(u.shape)
        gb = b.sim.state().reshape(u.shape[0], nz, 3 * ny, nx)
        for c in range(3):
            assert np.array_equal(gb[:, :, c * ny:(c + 1) * ny], ga)
    finally:
        a.close()
        b.close()
