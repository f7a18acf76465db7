"""Weight and bias gradients at the edges of their tiles and z-chunks.

The weight-gradient kernel covers the x-y plane with 256-voxel tiles of width 32, 16 or 8 and
the planes with chunks.  These slabs leave tiles partly empty in x and y, take every tile
width, and end in a short chunk.  Inputs are the dyadic ones of tests/unet_dyadic.py; the cell
counts here are no powers of two, so the target is placed at (odd part of the cell count) times
a dyadic distance from the output, which makes every 2 (out - target) / n dyadic again.  Every
signal is then exact and only the final FP32 sums over voxels differ: relative 1e-5, as in
tests/test_gpu_unet.py.
"""
import numpy as np
import pytest

import unet_dyadic as D
from oracle import unet_ref as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 4), (4, 8, 24), (4, 32, 40), (4, 16, 40), (28, 16, 32)])
def test_weight_gradient_at_tile_edges(shape):
    import torch
    from paper_2210_15668_amd import ferrox
    theta, x = D.params(50), D.inputs(51, shape)
    odd = int(np.prod(shape))
    while odd % 2 == 0:
        odd //= 2
    tgt = U.forward(theta, x, rnd=D.bf16) - odd * D.target(52, shape)
    assert np.array_equal(tgt.astype(np.float32).astype(np.float64), tgt)
    net = ferrox.UNet(shape[2], shape[1], shape[0], train=True)
    net.set_params(theta.astype(np.float32))
    net.set_input(x.astype(np.float32))
    loss, g = net.loss_grad(torch.from_numpy(tgt.astype(np.float32)).cuda())
    net.close()
    L_ref, g_ref = U.gradient(theta, x, tgt, rnd=D.bf16, grnd=D.bf16)
    assert abs(loss - L_ref) <= 1e-6 * L_ref
    p_gpu, p_ref = U.unpack(g.astype(np.float64)), U.unpack(g_ref)
    for name in ["head"] + [l[0] for l in U.LAYERS][::-1]:
        for part in (0, 1):
            a, b = p_gpu[name][part].ravel(), p_ref[name][part].ravel()
            assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b), (name, part)
            assert np.abs(a - b).max() <= 1e-5 * np.abs(b).max(), (name, part)
