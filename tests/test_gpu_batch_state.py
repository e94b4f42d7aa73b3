"""States of uneven batches in and out: every block's time step and fields bit for bit
those of the same block in a context of its own, from host and device memory (also off a
double's alignment), in both precisions; blocks smaller than a wavefront, of padded and
unpadded cell counts, fewer and more blocks than workgroups would be launched for one.
"""
import numpy as np
import pytest

from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_parity import random_mhd

pytestmark = pytest.mark.gpu

SETS = {"one": [(40, 24, 33)], "tiny": [(1, 1, 2), (3, 1, 1), (5, 7, 2)] * 3,
        "uneven": [(16, 16, 16), (33, 9, 20), (64, 48, 10), (2, 2, 2)], "many": [(4, 5, 3), (8, 4, 2)] * 150}


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("name", list(SETS))
def test_batch_state_round_trip(name, prec):
    import torch

    shapes = SETS[name]
    scheme = dict(recon="dc", riemann="hlle", integ="vl2", prec=prec)
    states = [random_mhd(sh, b % 7) for b, sh in enumerate(shapes)]
    lengths = [tuple(v / max(sh) for v in sh) for sh in shapes]
    dts, rows, alone = [], [], {}
    for b, (sh, L) in enumerate(zip(shapes, lengths)):
        if (sh, b % 7) not in alone:
            sim = B.Sim(sh, L, scheme=scheme)
            sim.set_state(states[b])
            alone[sh, b % 7] = sim.dt_cfl(), sim.state()
            sim.close()
        dts.append(alone[sh, b % 7][0])
        rows.append(alone[sh, b % 7][1])
    dts, ref, flat = np.array(dts), np.concatenate(rows), np.concatenate(states)
    bt = B.Batch(shapes, lengths, scheme=scheme)
    try:
        shifted = torch.zeros(flat.nbytes + 8, dtype=torch.uint8, device="cuda:0")
        shifted[4:-4] = torch.from_numpy(flat).view(torch.uint8).to("cuda:0")
        back = torch.zeros_like(shifted)
        dev = torch.from_numpy(flat).to("cuda:0")
        for put in (lambda: bt.set_state(states), lambda: bt.set_state(dev),
                    lambda: B.mhd_batch_set_state(bt.ctx, shifted.data_ptr() + 4, True)):
            bt.set_state(np.ones_like(flat))
            put()
            assert np.array_equal(bt.dt_cfl(), dts)
            assert np.array_equal(bt.state(), ref)
            assert np.array_equal(bt.state(device=True).cpu().numpy(), ref)
            B.mhd_batch_get_state(bt.ctx, back.data_ptr() + 4, True)
            torch.cuda.synchronize()
            assert np.array_equal(back[4:-4].cpu().numpy().view(np.float64), ref)
    finally:
        bt.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 7, 2), (64, 48, 10), (256, 130, 129)])
def test_device_state_as_host_state(shape, prec):
    """One grid: a state from device memory (also off a double's alignment) gives the bits
    and the time step of the same state from host memory, which goes another way (the last
    grid has more cells than one pass of its workgroups)."""
    import torch

    st = random_mhd(shape, 2)
    sim = B.Sim(shape, scheme=dict(recon="dc", riemann="hlle", integ="vl2", prec=prec))
    try:
        sim.set_state(st)
        dt, ref = sim.dt_cfl(), sim.state()
        shifted = torch.zeros(st.nbytes + 8, dtype=torch.uint8, device="cuda:0")
        shifted[4:-4] = torch.from_numpy(np.ascontiguousarray(st).reshape(-1)).view(torch.uint8).to("cuda:0")
        dev = torch.from_numpy(np.ascontiguousarray(st).reshape(-1)).to("cuda:0")
        for put in (lambda: sim.set_state(dev), lambda: B.mhd_set_state(sim.ctx, shifted.data_ptr() + 4, True)):
            sim.set_state(np.ones_like(st))
            put()
            assert sim.dt_cfl() == dt
            assert np.array_equal(sim.state(), ref)
    finally:
        sim.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32_bulk"])
@pytest.mark.parametrize("nd,shape", [(1, (1, 1, 1)), (3, (13, 11, 7)), (16, (65, 8, 9))])
def test_device_dust_state_as_host_state(nd, shape, prec):
    """The same for gas and dust, species below their floor among them."""
    import torch

    st, ts = I.dust_drift(shape=shape, nd=nd, seed=2, noise=0.3)
    st = np.ascontiguousarray(st, dtype=np.float64).reshape(-1)
    n = int(np.prod(shape))
    st[4 * n] = 0.0  # one dust cell below its floor
    sim = B.Sim(shape, physics=dict(eos="isothermal_hydro", tstop=ts),
                scheme=dict(recon="plm", riemann="hlle", integ="imex2p", prec=prec))
    try:
        sim.set_state(st)
        dt, ref = sim.dt_cfl(), sim.state()
        shifted = torch.zeros(st.nbytes + 8, dtype=torch.uint8, device="cuda:0")
        shifted[4:-4] = torch.from_numpy(st).view(torch.uint8).to("cuda:0")
        dev = torch.from_numpy(st).to("cuda:0")
        for put in (lambda: sim.set_state(dev), lambda: B.mhd_set_state(sim.ctx, shifted.data_ptr() + 4, True)):
            sim.set_state(np.ones_like(st))
            put()
            assert sim.dt_cfl() == dt
            assert np.array_equal(sim.state(), ref)
    finally:
        sim.close()
