"""FP64 states of a batch out by a copy per block (a single one, or large ones) and by the
storing kernel, without and with padding between the blocks.  The time steps of blocks with
more and fewer CFL partials than one wave takes in a round (512)."""
import numpy as np
import pytest

from paper_2608_14048_amd import binding as B
from tests.test_gpu_parity import random_mhd

pytestmark = pytest.mark.gpu

SETS = {"one odd": [(13, 7, 5)], "dense": [(16, 8, 4), (8, 8, 8)], "padded after": [(16, 8, 4), (5, 3, 7)],
        "padded": [(5, 3, 7), (16, 8, 4), (8, 8, 8), (3, 3, 3)], "copied": [(131, 127, 129), (129, 131, 128)],
        "partials": [(64, 64, 33), (64, 64, 32)]}


@pytest.mark.parametrize("name", list(SETS))
def test_states_in_and_out(name):
    import torch

    shapes = SETS[name]
    scheme = dict(recon="dc", riemann="hlle", integ="vl2")
    states = [random_mhd(sh, b) for b, sh in enumerate(shapes)]
    flat = np.concatenate(states)
    bt = B.Batch(shapes, scheme=scheme)
    try:
        bt.set_state(torch.from_numpy(flat).to("cuda:0"))
        for b, (sh, L) in enumerate(zip(bt.shapes, bt.lengths)):
            s = B.Sim(sh, L, scheme=scheme)
            s.set_state(states[b])
            assert bt.dt_cfl()[b] == s.dt_cfl()
            s.close()
        assert np.array_equal(bt.state(), flat)
        assert np.array_equal(bt.state(device=True).cpu().numpy(), flat)
        raw = torch.zeros(flat.nbytes + 16, dtype=torch.uint8, device="cuda:0")
        for off in (4, 8):  # off a double's alignment, and off two doubles'
            raw.zero_()
            B.mhd_batch_get_state(bt.ctx, raw.data_ptr() + off, True)
            torch.cuda.synchronize()
            got = raw.cpu().numpy()
            assert np.array_equal(got[off:off + flat.nbytes].view(np.float64), flat)
            assert not got[:off].any() and not got[off + flat.nbytes:].any()
    finally:
        bt.close()
