"""The convolution and gradient kernels on grids that do not fill their voxel blocks
(16 x 4 x 8 and 16 x 4 x 4): single rows and planes, remainders in y and z, several
blocks along x, more blocks than workgroups.

Both sides round the same operands to BF16, so what is left is FP32 accumulation order
and the few hidden activations it rounds the other way: at most a BF16 step (2^-8) of
single activations, 2e-2 of the largest output and 1e-2 of a layer's gradient norm.
"""
import numpy as np
import pytest

from oracle import closure as C
from paper_2608_14048_amd import binding as B
from paper_2608_14048_amd import inputs as I
from tests.test_gpu_closure import dev, emulated_acts, emulated_backward, random_params

pytestmark = pytest.mark.gpu


def rough_state(shape, rng):
    full = tuple(reversed(shape))
    rho = rng.uniform(0.5, 1.5, full)
    v = [rng.normal(0, 0.5, full) for _ in range(3)]
    b = [rng.normal(0, 0.5, full) for _ in range(3)]
    return I.mhd_state(rho, *v, rng.uniform(0.6, 1.8, full), *b)


@pytest.mark.parametrize("shape", [(16, 1, 1), (16, 3, 9), (32, 5, 17), (48, 4, 4), (16, 9, 3), (16, 20, 420)])
def test_forward_and_gradients_on_ragged_blocks(shape):
    rng = np.random.default_rng(sum(shape))
    st = rough_state(shape, rng)
    L = tuple(v / max(shape) for v in shape)
    params = random_params(rng)
    w = C.primitives(st, shape).reshape(8, -1)
    f32 = lambda a: np.asarray(a, dtype=np.float32)  # noqa: E731
    mu, sd, sF, sE = f32(w.mean(axis=1)), f32(w.std(axis=1) + 1e-3), f32([1e-2, 2e-2, 2e-2, 2e-2, 3e-2]), 1e-2
    wU, wB = np.array([1.0, 2.0, 2.0, 2.0, 0.5]), 1.5
    cl = B.Closure(shape, L)
    try:
        cl.set_params(f32(C.pack(params)))
        cl.set_scales(mu, sd, sF, sE, f32(wU), wB)
        params = C.unpack(f32(C.pack(params)).astype(np.float64))
        x = C.normalised_input(st, shape, mu.astype(np.float64), sd.astype(np.float64))
        ref, acts = emulated_acts(params, x)
        out = cl.forward(dev(st)).cpu().numpy().reshape(ref.shape)
        assert np.abs(out - ref).max() < 2e-2 * np.abs(ref).max()
        assert np.abs(out - ref).mean() < 2e-3 * np.abs(ref).mean()

        dt, dx = 2e-3, tuple(L[a] / shape[a] for a in range(3))
        coarse = st + 1e-4 * rng.standard_normal(st.shape)
        target = st + 1e-4 * rng.standard_normal(st.shape)
        cl.zero_grad()
        for _ in range(2):  # gradients add up over samples
            loss = cl.accumulate(dev(st), dev(coarse), dev(target), dt)
        g = cl.grads().astype(np.float64) / 2
        s64, e64 = sF.astype(np.float64), float(np.float32(sE))
        pred = C.apply_closure(coarse, shape, ref, s64, e64, dt, dx)
        ref_loss = C.loss(pred, target, shape, wU, wB)
        assert abs(loss - ref_loss) <= 1e-3 * ref_loss
        grads = emulated_backward(params, acts, C.loss_grad_out(pred, target, shape, s64, e64, dt, dx, wU, wB))
        at = 0
        for l, (W, b) in enumerate(grads):
            for part in ((W, b) if l < 3 else (W,)):  # (the output biases are a null direction)
                r = part.reshape(-1)
                a = g[at:at + r.size]
                rel = np.linalg.norm(a - r) / np.linalg.norm(r)
                print(f"  {shape} layer {l} {part.shape}: relative L2 {rel:.2e}", flush=True)
                assert rel < 1e-2
                at += r.size
    finally:
        cl.close()
