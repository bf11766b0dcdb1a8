"""The convolution variants that a large batch takes (tall tiles, all channels
in one workgroup), on grids whose three resolutions leave ragged last tiles.

Tile shapes only regroup the outputs: each is the same sum in the same order, so
an image's fields are the same bits in a batch as alone.  For the gradients every
target but the first and the last image's is the network's own output: those
images' output gradients are zero, and the batch gradient is the mean of two
images' times 2 / B.  B is a power of two, so that factor is exact and the
element-wise bounds of the small-batch tests hold as they are.
"""
import numpy as np
import pytest

from oracle import cnn as ocnn
from test_gpu_cnn import _setup, check_forward, check_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,B,in_ch", [(132, 52, 256, 1), (140, 36, 256, 3)])
def test_large_batch_matches_single_images(nx, ny, B, in_ch):
    import torch
    k = 10
    s = _setup(nx, ny, B, k, seed=nx, in_ch=in_ch)
    net, op, eps, eps_d = s[:4]
    eim, eim_d = s[4:] if in_ch == 3 else (None, None)

    def fields(sl):
        return net.predict(eps_d[sl], eim=None if eim is None else eim_d[sl])

    U = fields(slice(0, B))
    for b in (0, 1, B // 2 + 1, B - 1):
        assert torch.equal(fields(slice(b, b + 1))[0], U[b]), b

    ends = [0, B - 1]
    rng = np.random.default_rng(nx + 1)
    tgt = U.clone()
    two = ((rng.standard_normal((2, k, nx * ny)) + 1j * rng.standard_normal((2, k, nx * ny)))
           * 0.1).astype(np.complex64)
    tgt[ends] = torch.tensor(two, device="cuda").reshape(tgt[ends].shape)
    loss, g = net.grad(eps_d, tgt, eim=eim_d)

    class Ends:   # the two images' activations, as check_forward reads them
        layers = staticmethod(net.layers)

        @staticmethod
        def activation(li, n):
            return net.activation(li, B)[ends]

    out, cache = check_forward(Ends, op, eps[ends], k, 2,
                               eim=None if eim is None else eim[ends], Ugpu=U[ends].cpu().numpy())
    lo, dout = ocnn.mse(out, ocnn.fields_to_channels(two.astype(np.complex128), ny, nx))
    assert abs(loss * (B // 2) - lo) < 1e-4 * lo, (loss, lo)
    check_grads(net, op, cache, dout, k, np.asarray(g, np.float64) * (B // 2))
