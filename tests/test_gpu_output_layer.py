"""The output layer of 5 points and more on both sides of each line between its two
kernels (short sums, many outputs, many points), against the oracle."""
import numpy as np
import pytest

from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    c = nnc.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("K,m,B", [(64, 10, 5), (64, 10, 16), (64, 10, 17), (64, 256, 17), (64, 257, 17), (65, 512, 63),
                                   (130, 513, 29), (130, 513, 33), (512, 1024, 70), (512, 1025, 5), (512, 1025, 20),
                                   (2100, 1100, 21), (2100, 1100, 25), (4096, 3000, 5), (300, 4200, 9)])
def test_output_layer(ctx, prec, K, m, B):
    dims, acts = (9, K, m), ["tanh", "identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=51, bias_scale=0.2)
    X, _ = datagen.points(dims[0], m, B, seed=52)
    net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=B)
    g = net.eval_g(X).cpu().numpy()
    net.destroy()
    for b in (0, 3, B - 1):
        ref = O.nn(Ws, bs, acts, X[b])
        assert np.linalg.norm(g[b] - ref) < TOL[prec] * np.linalg.norm(ref), b
