"""PPM beside a cell that is not finite: Colella and Woodward's conditions as they are
written make the face states on both sides of such a cell bad (a false comparison leaves a
parabola's edges alone), so one stage makes exactly the cells that share a face with it bad,
whatever the direction of the flow; and a cell two away, whose face states stay finite, gets
the values those conditions give.  The second is taken along each axis from a supersonic
flow of constant velocity and pressure, where the mass flux is the upwind density times the
velocity: the density after a step follows from the reconstruction alone (numpy, FP64; a few
roundings of each precision allowed)."""
import numpy as np
import pytest

from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_ppm_limits import stepped_state

pytestmark = pytest.mark.gpu


def sim(shape, length, riemann, prec):
    return B.Sim(shape, length, scheme=dict(recon="ppm", riemann=riemann, integ="euler1", prec=prec))


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("riemann", ["hlld", "hlle"])
@pytest.mark.parametrize("shape", [(16, 12, 10), (33, 18, 7), (40, 9, 12), (7, 5, 40)])
def test_a_bad_cell_reaches_its_neighbours(shape, riemann, prec):
    nx, ny, nz = shape
    s = sim(shape, (1.0, 1.0, 1.0), riemann, prec)
    try:
        for field in range(8):
            # near the middle, and in a corner (periodic neighbours, other tiles)
            for at in ((nx // 2, ny // 2, nz // 2), (0, ny - 1, 0)):
                st = stepped_state(shape, 3)
                s.set_state(st)
                dt = s.dt_cfl()
                st.reshape(8, nz, ny, nx)[field, at[2], at[1], at[0]] = np.nan
                s.set_state(st)
                s.step(dt)
                bad = ~np.isfinite(s.state().reshape(8, nz, ny, nx)[:5])
                seeds = {at}
                if field >= 5:  # a face value enters the cells on both its sides
                    low = list(at)
                    low[field - 5] -= 1
                    seeds.add(tuple(low))
                want = np.zeros((nz, ny, nx), dtype=bool)
                for c in seeds:
                    for d in ((0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)):
                        want[(c[2] + d[2]) % nz, (c[1] + d[1]) % ny, (c[0] + d[0]) % nx] = True
                for q in range(5):
                    assert np.array_equal(bad[q], want), (field, at, q, bad[q].sum(), want.sum())
    finally:
        s.close()


def upwind_states(a):
    """The state on the high face of every cell of a periodic line (from its own parabola)."""
    am, ap = np.roll(a, 1), np.roll(a, -1)
    dm, dp, c = a - am, ap - a, 0.5 * (ap - am)
    with np.errstate(invalid="ignore"):
        lim = np.minimum(np.abs(c), 2 * np.minimum(np.abs(dm), np.abs(dp)))
        m = np.where(dm * dp > 0, np.copysign(lim, c), 0.0)
        iface = 0.5 * (a + ap) - (np.roll(m, -1) - m) / 6.0  # between a cell and the next
        lo, hi = np.roll(iface, 1), iface
        flat = (hi - a) * (a - lo) <= 0
        da, a6 = hi - lo, 6 * (a - 0.5 * (lo + hi))
        return np.where(flat, a, np.where(-da * da > da * a6, 3 * a - 2 * lo, hi))


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-14), ("fp32_bulk", 2e-6)])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_cells_two_away_follow_the_conditions(axis, prec, tol):
    n = 48
    shape = tuple(n if a == axis else 1 for a in range(3))
    length = tuple(1.0 if a == axis else 1.0 / n for a in range(3))
    full = shape[::-1]
    rng = np.random.default_rng(4)
    s = sim(shape, length, "hlle", prec)
    try:
        for k in range(6):
            rho = np.cumsum(rng.uniform(0.02, 0.1, n))[::1 - 2 * (k % 2)]  # a ramp up or down: few slopes are zero
            rho = np.float32(1.0 + np.where(rng.random(n) < 0.2, 0.5 * rho, rho)).astype(np.float64)
            v = [np.full(full, 4.0 if a == axis else 0.0) for a in range(3)]
            zero = np.zeros(full)
            st = I.mhd_state(rho.reshape(full), *v, np.full(full, 0.5), zero, zero, zero)
            s.set_state(st)
            dt = 0.5 * s.dt_cfl()
            b = int(rng.integers(n))
            rho[b] = np.nan
            st[b] = np.nan
            s.set_state(st)
            s.step(dt)
            got = s.state()[:n]
            flux = 4.0 * upwind_states(rho)
            want = rho - dt * n * (flux - np.roll(flux, 1))
            # (the high face of the cell below the bad one and the bad one's own are bad)
            near = [(b - 1) % n, b, (b + 1) % n]
            assert np.isnan(got[near]).all()
            keep = np.setdiff1d(np.arange(n), near)
            assert np.isfinite(want[keep]).all()
            err = np.abs(got[keep] - want[keep]).max() / np.nanmax(rho)
            assert err <= tol, (err, keep[np.abs(got[keep] - want[keep]).argmax()], b)
    finally:
        s.close()
