"""Device KKT solve of matrices whose neighbouring unknowns are strongly coupled:
a smooth (Gaussian) kernel on [0, 1] plus a small multiple of the identity, whose
16 x 16 diagonal blocks are as badly conditioned as the whole.  Cholesky factors
them without trouble, and its residual does not know the condition number.  Also
pivots below the range in which their reciprocals are finite."""
import numpy as np
import pytest

from paper_2509_22462_amd import nnc

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


def solve(ctx, M, r):
    import torch
    B, n = r.shape
    kkt = nnc.nnc_kkt_create(ctx.h, n, B)
    H, rd = (torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (M, r))
    dx = torch.full((B, n), np.nan, dtype=torch.float64, device="cuda")
    info = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    rc = nnc.nnc_kkt_solve(ctx.h, kkt, B, H.data_ptr(), None, None, None, None, rd.data_ptr(), dx.data_ptr(),
                           info.data_ptr())
    assert rc == nnc.NNC_OK, nnc.nnc_last_error(ctx.h)
    torch.cuda.synchronize()
    nnc.nnc_kkt_destroy(ctx.h, kkt)
    return dx.cpu().numpy(), info.cpu().numpy()


def kernel(n, eps, width=0.02):
    t = np.linspace(0.0, 1.0, n)
    return np.exp(-0.5 * ((t[:, None] - t[None, :]) / width) ** 2) + eps * np.eye(n)


# conditions 1e7 to 1e12; one panel, a ragged last one, and many
@pytest.mark.parametrize("n", [64, 130, 256, 784])
def test_positive_definite_is_accepted(ctx, n):
    eps = (1e-6, 1e-8, 1e-10, 1e-11)
    M = np.stack([kernel(n, e) for e in eps])
    r = np.random.default_rng(n).standard_normal((len(eps), n))
    for m in M:
        np.linalg.cholesky(m)  # positive definite in FP64
    x, info = solve(ctx, M, r)
    assert info.tolist() == [0] * len(eps)


def backward_error(M, x, r):
    return np.linalg.norm(M @ x - r) / (np.linalg.norm(M, 2) * np.linalg.norm(x) + np.linalg.norm(r))


# The residual of a backward stable solve is some units of 2^-53 of |M| |x|
# whatever the condition; each of the n / 16 blocks adds its own, at random.
@pytest.mark.parametrize("B", [1, 5])
@pytest.mark.parametrize("n", [40, 64, 130, 256, 784, 2048])
def test_residual_is_independent_of_the_condition(ctx, n, B):
    eps = np.logspace(-6, -11, B) if B > 1 else np.array([1e-9])
    M = np.stack([kernel(n, e) for e in eps])
    r = np.random.default_rng(n).standard_normal((B, n))
    x, info = solve(ctx, M, r)
    assert np.all(info == 0)
    for b in range(B):
        assert backward_error(M[b], x[b], r[b]) < 4 * np.sqrt(n / 16) * 2.0 ** -53, eps[b]


@pytest.mark.parametrize("n", [1, 20, 70])
def test_subnormal_pivots(ctx, n):
    """Diagonal systems down to the least normal numbers and below: x = r / d, d
    and r exact, to a few roundings."""
    d = np.logspace(-307, -314, n)
    x, info = solve(ctx, np.diag(d)[None], 3.0 * d[None])
    assert info.tolist() == [0]
    assert np.max(np.abs(x / ((3.0 * d) / d) - 1.0)) < 8 * 2.0 ** -53
