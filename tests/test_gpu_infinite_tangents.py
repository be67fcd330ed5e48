"""Tangents past the FP32 range: an infinite tangent times a weight or another
tangent is infinite, on packed operands as in the row-major products (which
forcing a tiling brings back), and NaN only where the product is."""
import numpy as np
import pytest

from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    c = nnc.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


# the value of the other weights: exact in BF16 (two of its three parts are
# zero), with three parts, and zero; K split or not
@pytest.mark.parametrize("weight", [0.5, 1.0 / 3.0, 0.0])
@pytest.mark.parametrize("width", [8, 64, 1500])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_tangents(ctx, weight, width, sign):
    n, j, u = 20, 7, 3
    dims = (n, width, width, width, 2)
    W1 = np.full((width, n), 0.25)
    W1[:, j] = sign * 1e25
    W2 = np.full((width, width), 0.25)
    W2[u] = 1e14  # T_2[u, j] = 1e39 width: infinite in FP32
    W3 = np.full((width, width), weight)
    W4 = np.full((2, width), 1.0)
    bs = [np.zeros(width), np.full(width, 0.5), np.full(width, 0.5), np.zeros(2)]
    acts = ["tanh", "tanh", "tanh", "identity"]
    X, Lam = np.zeros((1, n)), np.ones((1, 2))
    net = ctx.net(dims, acts, [W1, W2, W3, W4], bs, prec="fp32", max_points=1)
    net.set_hess_method("layersum")
    code = nnc.PREC_CODES["fp32"]
    H = net.eval_hess_lag(X, Lam).cpu().numpy()[0]
    try:
        assert nnc.nnc_set_gemm_config(ctx.h, code, 3) == nnc.NNC_OK
        R = net.eval_hess_lag(X, Lam).cpu().numpy()[0]
    finally:
        nnc.nnc_set_gemm_config(ctx.h, code, -1)
    net.destroy()
    assert np.any(~np.isfinite(R))
    assert np.array_equal(np.isnan(H), np.isnan(R))
    assert np.array_equal(np.isinf(H), np.isinf(R))
    assert np.array_equal(np.sign(H[np.isinf(H)]), np.sign(R[np.isinf(R)]))
    if weight and weight <= 0.5 and width == 64 and sign > 0:
        # nothing padded or saturated; every tangent and weight positive, every s negative
        assert np.all(H[j] == -np.inf) and np.all(H[:, j] == -np.inf)
    ok = np.isfinite(R)
    assert np.allclose(H[ok], R[ok], rtol=1e-4)
