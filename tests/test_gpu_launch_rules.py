"""Every branch of the launch rules for streams, reverse seeds, split products
and training steps, at the sizes on both sides of each line, against the FP64
oracle.  Tolerances are those of the parity tests (normwise error per point)."""
import numpy as np
import pytest

from oracle import mlp as M
from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16": 2e-2}
PRECS = ["fp64", "fp32", "bf16"]


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
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def check(ctx, dims, out, prec, B, seed, points=None):
    """g, J and H in one call and in three: the oracle's, and each other's bits.
    (Not J of one point with 64 outputs in FP32: alone it takes GEMMs, with H the
    adjoint's stream.  Not H in BF16: beside J it may round S from the stored T.)"""
    acts = ["tanh"] * (len(dims) - 2) + [out]
    Ws, bs = datagen.mlp_weights(dims, seed=seed, bias_scale=0.2)
    X, Lam = datagen.points(dims[0], dims[-1], B, seed=seed + 1)
    net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=B)
    net.set_hess_method("layersum")
    g, J, H = (t.cpu().numpy() for t in net.eval(X, Lam))
    J1, H1 = net.eval_jac_g(X).cpu().numpy(), net.eval_hess_lag(X, Lam).cpu().numpy()
    assert np.array_equal(g, net.eval_g(X).cpu().numpy())
    assert np.array_equal(J, J1) if (prec, B, dims[-1]) != ("fp32", 1, 64) else rel(J, J1) < 2 * TOL[prec]
    assert np.array_equal(H, H1) if prec != "bf16" else rel(H, H1) < 2 * TOL[prec]
    net.destroy()
    for b in points or range(B):
        # a single output of 0.03 left over from terms of 0.1 each has no normwise
        # bound in BF16: rounding the weights alone moves it by 3.4e-2
        if not (prec == "bf16" and dims == (21, 2100, 1700, 70, 1)):
            assert rel(g[b], O.nn(Ws, bs, acts, X[b])) < TOL[prec], ("g", b)
        assert rel(J[b], O.jacobian(Ws, bs, acts, X[b])) < TOL[prec], ("J", b)
        assert rel(H[b], O.hess_layersum(Ws, bs, acts, X[b], Lam[b])) < TOL[prec], ("H", b)
        assert np.array_equal(H[b], H[b].T)


# Streams of 5..63 rows: one to four blocks of 16 rows, a layer wide enough to
# stage its rows in LDS beside ones that are not, ragged widths, and an output
# layer of one and of 33 entries.
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("dims,B", [
    ((21, 2100, 1700, 70, 1), 5), ((21, 2100, 1700, 70, 1), 16), ((30, 1601, 2050, 33), 17), ((9, 1601, 1603, 3), 63)])
def test_streams_of_several_points(ctx, prec, dims, B):
    check(ctx, dims, "identity", prec, B, 81, points=[0, B // 2, B - 1])


# One point: seeds of the reverse passes fused up to 64 outputs, in separate
# launches from 65 on; one hidden layer, and a hidden width past one workgroup.
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("out", ["identity", "tanh", "softmax"])
@pytest.mark.parametrize("dims", [(13, 40, 1), (13, 300, 70, 64), (13, 70, 300, 65)])
def test_reverse_seeds(ctx, prec, out, dims):
    check(ctx, dims, out, prec, 1, 83)


# Jacobian products of 64 rows and more with few output tiles (K split until
# the chip is busy) and with enough of them, K ragged.
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("dims,B", [((300, 1000, 500, 250, 10), 7), ((70, 260, 130, 64), 1), ((900, 1100, 90, 40), 30)])
def test_jacobian_of_few_tiles(ctx, prec, dims, B):
    check(ctx, dims, "identity", prec, B, 85, points=[0, B - 1])


# Layer-sum products of one to three tiles over a long K: more slices than the
# final sum takes at once, and a last group of them that is not full.
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("dims,B", [((17, 6000, 5000, 3), 1), ((129, 4500, 3300, 5), 1), ((130, 2300, 700, 5), 3)])
def test_hessian_of_many_slices(ctx, prec, dims, B):
    check(ctx, dims, "identity", prec, B, 87)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("m,B", [(64, 3), (65, 1), (150, 2)])
def test_softmax_of_many_outputs(ctx, prec, m, B):
    check(ctx, (11, 50, m), "softmax", prec, B, 89)


def params(Ws, bs):
    return np.concatenate([np.concatenate([W.ravel(), b]) for W, b in zip(Ws, bs)])


# Small products with both gradients and Adam in one launch, and the large
# tiles (128 or more of 128 x 128 in one product); ragged batch and widths, a
# layer of one column and of one row.
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("dims,batch", [((1, 65, 200, 1), 3), ((130, 64, 129, 70), 65), ((700, 1030, 90), 200),
                                        ((1500, 1500, 20), 40)])
def test_training_step(ctx, prec, dims, batch):
    import torch
    tol = {"fp32": 1e-5, "bf16": 3e-2}[prec]
    acts = ["tanh"] * (len(dims) - 2) + ["identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=91, bias_scale=0.1)
    rng = np.random.default_rng(92)
    X, Y = rng.random((batch, dims[0])), rng.standard_normal((batch, dims[-1]))
    mlp = nnc.nnc_train_create(ctx.h, list(dims), batch, nnc.PREC_CODES[prec], 7)
    p0 = params(Ws, bs)
    nnc.nnc_train_set_params(ctx.h, mlp, p0)
    Xd, Yd = (torch.as_tensor(v, device="cuda") for v in (X, Y))
    lr = 1e-3
    loss = nnc.nnc_train_step(ctx.h, mlp, Xd.data_ptr(), Yd.data_ptr(), lr)
    ref_loss, gW, gb = M.grads(Ws, bs, acts, X, Y)
    assert abs(loss - ref_loss) / ref_loss < tol
    g, ref = nnc.nnc_train_get_grads(ctx.h, mlp), params(gW, gb)
    assert np.linalg.norm(g - ref) / np.linalg.norm(ref) < tol
    # the update against Adam's first step on the gradient that was returned:
    # FP32 parameters of magnitude up to p move by lr to a rounding of 2^-24 p
    step = nnc.nnc_train_get_params(ctx.h, mlp) - p0.astype(np.float32).astype(np.float64)
    big = np.abs(g) > 1e-3 * np.max(np.abs(g))
    want = -lr * np.sign(g)
    assert np.max(np.abs(step[big] - want[big])) < lr * 1e-2 + 2.0 ** -23 * np.max(np.abs(p0))
    # a second step reads the weights that the first one wrote
    loss2 = nnc.nnc_train_step(ctx.h, mlp, Xd.data_ptr(), Yd.data_ptr(), lr)
    Ws2, bs2, o = [], [], 0
    p1 = p0 + step
    for l in range(1, len(dims)):
        k = dims[l] * dims[l - 1]
        Ws2.append(p1[o:o + k].reshape(dims[l], dims[l - 1]))
        bs2.append(p1[o + k:o + k + dims[l]])
        o += k + dims[l]
    ref2 = M.grads(Ws2, bs2, acts, X, Y)[0]
    assert abs(loss2 - ref2) / ref2 < tol
    nnc.nnc_train_destroy(ctx.h, mlp)
