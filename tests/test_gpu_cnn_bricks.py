"""The network's brick kernels at grids whose bricks overhang in y or z and at one-brick grids."""
import numpy as np
import pytest

from oracle import cnn
from test_gpu_cnn import FWD_TOL, GRAD_TOL, case, rel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1306_1821_amd.binding import CNN, cnn_flatten, cnn_unflatten  # noqa: E402


# 4: a quarter brick; 12: y and z overhang; 20: a full brick and an overhang; 36: more
@pytest.mark.parametrize("n", [4, 12, 20, 36])
def test_overhanging_bricks_match_oracle(n):
    """Forward and gradients with the end-to-end tolerances of the other network tests; the
    layers' weight gradients from the device's own activations and output gradients to the
    float32 accumulation bound 1e-4 used there."""
    params, x, target = case(n, 300 + n)
    net = CNN(params)
    inputs = np.moveaxis(x, -1, 0)
    xx, tt = (a.astype(np.float32).astype(np.float64) for a in (x, target))
    mu, s, cache = cnn.forward(params, xx, bf=True)
    got = net.forward(inputs)
    assert rel(got[0].cpu().numpy(), mu) < FWD_TOL and rel(got[1].cpu().numpy(), s) < FWD_TOL
    g, loss = net.gradient(inputs, target)
    assert abs(loss - cnn.loss(mu, s, tt)) < 1e-4 * abs(loss)
    gl = cnn_unflatten(g)
    rl = cnn_unflatten(cnn_flatten(cnn.backward(params, cache, mu, s, tt, bf=True)).astype(np.float64))
    a_in = cnn.bf16(xx)
    for l in range(4):
        z, a, dz = net.layer_state(l, n)
        dW, db = cnn.conv_weight_grad(a_in, dz.reshape(n, n, n, -1))
        assert rel(gl[l][0], dW) < 1e-4 and rel(gl[l][1], db) < 1e-4, l
        if n > 4:  # a 4^3 gradient sums 64 voxels: rounding flips alone exceed the bound
            assert rel(gl[l][0], rl[l][0]) < GRAD_TOL and rel(gl[l][1], rl[l][1]) < GRAD_TOL, l
        if a is not None:
            a_in = a.reshape(n, n, n, -1)
    net.close()


@pytest.mark.parametrize("n", [4, 8, 12, 20])
def test_last_layer_every_voxel(n):
    """The last layer from the device's own activations, in training (products in the order of
    the taps) and alone (its taps in pairs, its three y taps in the matrix rows), against a
    float64 convolution with the weights rounded to bfloat16: each output within the bound of
    a float32 sum of 433 terms, 434 2^-24 sum |w a|."""
    params, x, target = case(n, 700 + n)
    net = CNN(params)
    inputs = np.moveaxis(x, -1, 0)
    net.gradient(inputs, target)
    a, z = net.layer_state(2, n)[1].reshape(n, n, n, -1), net.layer_state(3, n)[0]
    alone = np.stack([o.cpu().numpy().astype(np.float64).ravel() for o in net.forward(inputs)], -1)
    W, b = params[3]
    W = cnn.bf16(W)
    want = cnn.conv(a, W, b).reshape(-1, 2)
    size = cnn.conv(np.abs(a), np.abs(W), np.abs(b)).reshape(-1, 2)
    assert np.all(np.abs(z - want) <= 434 * 2.0 ** -24 * size)
    assert np.all(np.abs(alone - want) <= 434 * 2.0 ** -24 * size)
    net.close()
