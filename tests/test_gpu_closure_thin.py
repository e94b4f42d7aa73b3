"""The closure on grids of few planes or few rows, whose convolutions take flat voxel blocks
(32 rows of a plane, or a row of 32 planes) where 4 x 8 blocks would be mostly padding:
against the reference as on other grids, and bit for bit the planes (rows) of the same
pattern repeated until 4 x 8 blocks are taken."""
import numpy as np
import pytest

from paper_2608_14048_amd import binding as B
from tests.test_gpu_closure import dev, random_params
from tests.test_gpu_closure_blocks import rough_state
from tests.test_gpu_closure_blocks import test_forward_and_gradients_on_ragged_blocks as against_reference
from oracle import closure as C

pytestmark = pytest.mark.gpu


# 275 and more blocks of 4 x 8 (two rounds of workgroups), remainders along the flat side
@pytest.mark.parametrize("shape", [(16, 1100, 1), (16, 1, 2201), (32, 2, 1100)])
def test_thin_grids_against_the_reference(shape):
    against_reference(shape)


@pytest.mark.parametrize("shape,axis", [((16, 1100, 1), 2), ((32, 555, 1), 2), ((16, 1, 2201), 1), ((48, 1, 750), 1)])
def test_thin_grid_equals_its_repetition(shape, axis):
    rng = np.random.default_rng(5)
    st = rough_state(shape, rng)
    params = C.pack(random_params(rng)).astype(np.float32)
    times = 8
    wide = tuple(v * (times if a == axis else 1) for a, v in enumerate(shape))
    L = tuple(v / max(shape) for v in shape)
    u = st.reshape(8, *shape[::-1])
    rep = np.ascontiguousarray(np.repeat(u, times, axis=3 - axis))
    one = B.Closure(shape, L)
    many = B.Closure(wide, tuple(v * (times if a == axis else 1) for a, v in enumerate(L)))
    try:
        for cl in (one, many):
            cl.set_params(params)
        a = one.forward(dev(st)).cpu().numpy().reshape(18, *shape[::-1])
        b = many.forward(dev(rep.reshape(-1))).cpu().numpy().reshape(18, *wide[::-1])
        assert np.abs(a).max() > 0
        assert np.array_equal(b, np.repeat(a, times, axis=3 - axis))
    finally:
        one.close()
        many.close()
