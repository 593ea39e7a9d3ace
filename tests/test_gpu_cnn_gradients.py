"""Parameter gradients of the network on grids that end inside the cell tiles
of the weight-gradient kernel (8 x 8 x 4 cells in 3D, 8 x 32 in 2D), on the
smallest ones and on some of several tiles a split, against the bf16-operand
oracle."""
import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (12, 100), (132, 36), (256, 520), (4, 4, 4), (4, 40, 12), (12, 20, 28), (36, 8, 20), (52, 48, 44)]


def exact_case(shape):
    """A network and data whose bf16 operands do not depend on the order of
    FP32 sums: three weights of +-1 per output channel and small whole numbers,
    so that the sums that are rounded to bf16 are exact in FP32."""
    nd = len(shape)
    rng = np.random.default_rng(5)
    params = []
    for W, b in cnn.init_params(nd, 2):
        V = np.zeros_like(W).reshape(W.shape[0], -1)
        for row in V:
            row[rng.choice(row.size, 3, replace=False)] = rng.choice([-1.0, 1.0], 3)
        params.append((V.reshape(W.shape), rng.integers(0, 3, size=b.shape).astype(np.float64)))
    x = rng.integers(-3, 4, size=shape + (2,)).astype(np.float64)
    t = rng.integers(-8, 9, size=shape + (1,)).astype(np.float64)
    return params, x, t


def deviation(got, ref):
    return max(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
               for p, q in zip(got, ref) for a, b in zip(p, q))


@pytest.mark.parametrize("shape", SHAPES)
def test_gradients_on_ragged_grids(shape):
    from paper_2303_10499_amd import learned
    nd = len(shape)
    params, x, t = exact_case(shape)
    nz, nx, ny = shape[0], shape[-1], shape[1] if nd == 3 else 1
    net = learned.Net(nd, nx, ny, nz, train=True)
    net.set_params(learned.pack(params))
    net.forward(np.ascontiguousarray(x.reshape(-1, 2), dtype=np.float32))
    tf = np.ascontiguousarray(t.reshape(-1), dtype=np.float32)
    net.backward(tf)
    g1 = net.get_grads()
    net.backward(tf, accumulate=True)
    # the same sums again on top of the first: one FP32 rounding
    assert np.abs(net.get_grads() - 2 * g1).max() <= 2.0**-23 * np.abs(2 * g1).max()
    y, cache = cnn.forward(params, x, bf16=True)
    ref = cnn.backward(params, cache, y, t, bf16=True)
    # identical bf16 operands; only the FP32 order of the sums over cells differs
    assert deviation(learned.unpack(g1, nd), ref) <= 1e-5
