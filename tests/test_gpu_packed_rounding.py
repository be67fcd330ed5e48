"""Rounding of the FP32 layer-sum products on packed operands, on narrow networks,
where no long sum covers it: against the FP64 oracle their errors have no
preferred sign and are no larger than those of the row-major FP32 products
(which forcing a tiling brings back).  Weights are FP32 numbers, so no error
comes from storing them."""
import numpy as np
import pytest

from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

POINTS, NETS = 8, 24


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    c = nnc.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("hidden,out", [((16, 16, 16), "softmax"), ((40, 40), "tanh"), ((1, 1), "identity")])
def test_errors_have_no_sign_and_do_not_grow(ctx, hidden, out):
    dims = (24, *hidden, 5)
    acts = ["tanh"] * len(hidden) + [out]
    err = {-1: [], 3: []}  # packed, row-major 64 x 64 tiles
    mean = []
    for seed in range(NETS):
        Ws, bs = datagen.mlp_weights(dims, seed=400 + seed, bias_scale=0.2)
        Ws = [W.astype(np.float32).astype(np.float64) for W in Ws]
        X, Lam = datagen.points(dims[0], dims[-1], POINTS, seed=500 + seed)
        ref = [O.hess_layersum(Ws, bs, acts, x, lam) for x, lam in zip(X, Lam)]
        net = ctx.net(dims, acts, Ws, bs, prec="fp32", max_points=POINTS)
        net.set_hess_method("layersum")
        try:
            for cfg in err:
                assert nnc.nnc_set_gemm_config(ctx.h, nnc.PREC_CODES["fp32"], cfg) == nnc.NNC_OK
                for H, R in zip(net.eval_hess_lag(X, Lam).cpu().numpy(), ref):
                    err[cfg].append(np.linalg.norm(H - R) / np.linalg.norm(R))
                    if cfg == -1:  # relative size of the error along R itself
                        mean.append(np.sum((H - R) * R) / np.sum(R * R))
        finally:
            nnc.nnc_set_gemm_config(ctx.h, nnc.PREC_CODES["fp32"], -1)
            net.destroy()
    packed, rowmajor = (np.sqrt(np.mean(np.square(err[c]))) for c in (-1, 3))
    assert packed <= rowmajor, (packed, rowmajor)
    if max(hidden) < 6:  # row-major (equal above); one neuron's terms may cancel, so no bound on their relative error
        return
    # some six roundings of up to 2^-24 to either side, averaged over 192 Hessians
    # of independent points: below 1.5e-7 / sqrt(192) in all but one of 50
    assert abs(np.mean(mean)) < 2.5 * 1.5e-7 / np.sqrt(POINTS * NETS), np.mean(mean)
