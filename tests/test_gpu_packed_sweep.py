"""Layer-sum sweeps on packed operands: the shapes at which the packed tiles,
their K splits and the packing itself can go wrong, against the FP64 oracle and
against the row-major sweep of the same network (which forcing a tiling of the
row-major kernels brings back)."""
import numpy as np
import pytest

from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

# normwise error of H per precision, as the parity tests state them
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


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# (dims, points): one row block short of a tile and one past it, widths of one
# padded block and of odd sizes, an odd number of 64-element K blocks, a long K
# (K split), tangent rows that straddle 16-row blocks between points
SHAPES = [
    ((1, 64, 64, 3), 1),
    ((17, 65, 200, 5), 2),
    ((111, 130, 70, 4), 1),
    ((113, 64, 192, 300, 2), 3),
    ((16, 2000, 320, 4), 1),
    ((50, 320, 2000, 6), 5),
    ((40, 100, 90, 80, 7), 7),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("dims,B", SHAPES)
def test_packed_sweep_matches_oracle_and_row_major(ctx, prec, dims, B):
    acts = ["tanh"] * (len(dims) - 2) + ["identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=71, bias_scale=0.1)
    X, Lam = datagen.points(dims[0], dims[-1], B, seed=72)
    net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=B)
    net.set_hess_method("layersum")
    H = net.eval_hess_lag(X, Lam).cpu().numpy()
    assert np.array_equal(H, net.eval_hess_lag(X, Lam).cpu().numpy())
    code = nnc.PREC_CODES[prec]
    try:
        assert nnc.nnc_set_gemm_config(ctx.h, code, 3) == nnc.NNC_OK  # row-major 64 x 64 tiles
        Hr = net.eval_hess_lag(X, Lam).cpu().numpy()
    finally:
        assert nnc.nnc_set_gemm_config(ctx.h, code, -1) == nnc.NNC_OK
    assert np.array_equal(H, net.eval_hess_lag(X, Lam).cpu().numpy())  # back on packed operands
    for b in range(B):
        ref = O.hess_for(Ws, bs, acts, X[b], Lam[b])
        assert rel(H[b], ref) < TOL[prec], (b, rel(H[b], ref))
        assert rel(H[b], Hr[b]) < 2 * TOL[prec]
    net.destroy()


def test_packed_fp32_keeps_all_bits(ctx):
    """Elements spread over the exponent range (a hidden layer whose weights
    run over 20 decades along each row, against tangents that run the other way):
    weights rounded to FP32 once and about 20 roundings of 2^-24 in the sums stay
    below 2e-6; two parts instead of three (16 bits) would be off by 2^-17."""
    dims = (24, 96, 96, 3)
    acts = ["tanh", "tanh", "identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=73, bias_scale=0.1)
    X, Lam = datagen.points(dims[0], dims[-1], 1, seed=74)
    scale = 10.0 ** np.linspace(-10, 10, dims[1])
    Ws = [Ws[0] / 4.0, Ws[1] * scale[None, :], Ws[2]]
    # the first layer's outputs are small where the second's weights are large
    Ws[0] = Ws[0] / scale[:, None].clip(1.0)
    bs[0] = bs[0] / scale.clip(1.0)
    net = ctx.net(dims, acts, Ws, bs, prec="fp32", max_points=1)
    net.set_hess_method("layersum")
    H = net.eval_hess_lag(X, Lam).cpu().numpy()[0]
    ref = O.hess_for(Ws, bs, acts, X[0], Lam[0])
    assert rel(H, ref) < 2e-6, rel(H, ref)
    net.destroy()
