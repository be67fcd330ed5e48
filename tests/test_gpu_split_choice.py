"""K splits of products without a tuned row are chosen from the product alone:
the same points give the same bits whatever max_points the network was made for,
and before and after a split was forced and released."""
import numpy as np
import pytest

from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    c = nnc.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("method", ["for", "layersum"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("dims,B", [((21, 1509, 92, 1), 26), ((64, 300, 900, 64), 1), ((8, 2000, 70, 3), 9)])
def test_bits_do_not_depend_on_the_workspace(ctx, prec, method, dims, B):
    acts = ["tanh"] * (len(dims) - 2) + ["identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=31, bias_scale=0.2)
    X, Lam = datagen.points(dims[0], dims[-1], B, seed=32)
    code = nnc.PREC_CODES[prec]
    got = []
    for most in (B, 4 * B + 64):
        net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=most)
        net.set_hess_method(method)
        for forced in (False, True):
            if forced:
                assert nnc.nnc_set_gemm_ksplit(ctx.h, code, 3) == nnc.NNC_OK
                net.eval_hess_lag(X, Lam)
                assert nnc.nnc_set_gemm_ksplit(ctx.h, code, -1) == nnc.NNC_OK
            got.append((net.eval_jac_g(X).cpu().numpy(), net.eval_hess_lag(X, Lam).cpu().numpy()))
        net.destroy()
    for J, H in got[1:]:
        assert np.array_equal(J, got[0][0]) and np.array_equal(H, got[0][1])
    for b in (0, B - 1):
        R = O.hess_layersum(Ws, bs, acts, X[b], Lam[b])
        assert np.linalg.norm(got[0][1][b] - R) < TOL[prec] * np.linalg.norm(R)
