"""The panel kernels of the device KKT solve at the sizes where their blocking
can go wrong: whole panels, one row past them, the largest order, more systems
than panels, a matrix whose upper triangle holds no numbers, pivots at the ends
of the FP64 range and failures inside each 16-column sub-block."""
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


def solve(ctx, H, d, a, s, r):
    import torch
    B, n = r.shape
    kkt = nnc.nnc_kkt_create(ctx.h, n, B)
    t = [None if v is None else torch.as_tensor(np.ascontiguousarray(v), device="cuda") for v in (H, d, a, s, r)]
    p = [None if v is None else v.data_ptr() for v in t]
    dx = torch.full((B, n), np.nan, dtype=torch.float64, device="cuda")
    info = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    rc = nnc.nnc_kkt_solve(ctx.h, kkt, B, p[0], p[1], p[2], p[3], None, p[4], dx.data_ptr(), info.data_ptr())
    assert rc == nnc.NNC_OK, nnc.nnc_last_error(ctx.h)
    torch.cuda.synchronize()
    nnc.nnc_kkt_destroy(ctx.h, kkt)
    return dx.cpu().numpy(), info.cpu().numpy()


@pytest.mark.parametrize("n,B", [(128, 2), (129, 1), (191, 3), (320, 33), (1000, 2), (1025, 1), (2048, 1)])
def test_panels_and_lower_triangle(ctx, n, B):
    rng = np.random.default_rng(n)
    G = rng.standard_normal((B, n, n)) / np.sqrt(n)
    H = 0.5 * (G + G.transpose(0, 2, 1))
    d = 2.0 + rng.random((B, n))
    a = rng.standard_normal((B, n)) / np.sqrt(n)
    s = 3.0 * rng.random(B)
    r = rng.standard_normal((B, n))
    low = H.copy()
    low[:, np.triu(np.ones((n, n), dtype=bool), 1)] = np.nan  # only the lower triangle is read
    dx, info = solve(ctx, low, d, a, s, r)
    assert np.all(info == 0)
    for b in range(B):
        M = H[b] + np.diag(d[b]) + s[b] * np.outer(a[b], a[b])
        # backward stable: residual within a small multiple of n eps |M| |x|
        res = np.linalg.norm(M @ dx[b] - r[b])
        assert res < 1e-15 * n * (np.linalg.norm(M, 2) * np.linalg.norm(dx[b]) + np.linalg.norm(r[b])), (b, res)


@pytest.mark.parametrize("bad", [0, 15, 16, 47, 63, 64, 100, 127, 129])
def test_failure_in_each_sub_block(ctx, bad):
    n = 130
    d = np.ones((2, n))
    d[1, bad] = -1.0
    dx, info = solve(ctx, np.zeros((2, n, n)), d, None, None, np.ones((2, n)))
    assert info.tolist() == [0, bad + 1]
    assert np.allclose(dx[0], 1.0, rtol=0, atol=1e-15) and np.all(dx[1] == 0.0)


def test_pivots_over_the_fp64_range(ctx):
    """A diagonal system: every unknown is r / d to a few roundings of 2^-53."""
    n = 96
    d = np.logspace(-300, 300, n)[None, :]
    r = d * np.linspace(1.0, 2.0, n)
    dx, info = solve(ctx, np.zeros((1, n, n)), d, None, None, r)
    assert info[0] == 0
    assert np.max(np.abs(dx[0] / np.linspace(1.0, 2.0, n) - 1.0)) < 8 * 2.0 ** -53


@pytest.mark.parametrize("n,bad", [(1, 0), (1, None), (16, 15), (17, 16), (64, 0), (64, 63), (64, None), (65, 64)])
def test_one_panel_solved_or_zeroed(ctx, n, bad):
    """Up to 64 unknowns are factored and solved in one launch."""
    rng = np.random.default_rng(100 + n)
    G = rng.standard_normal((2, n, n)) / np.sqrt(n)
    H = 0.5 * (G + G.transpose(0, 2, 1))
    d = 3.0 + rng.random((2, n))
    if bad is not None:
        d[1, bad] = -50.0
    r = rng.standard_normal((2, n))
    dx, info = solve(ctx, H, d, None, None, r)
    assert info.tolist() == [0, 0 if bad is None else bad + 1]
    for b in range(2 if bad is None else 1):
        M = H[b] + np.diag(d[b])
        res = np.linalg.norm(M @ dx[b] - r[b])
        assert res < 1e-15 * max(n, 8) * (np.linalg.norm(M, 2) * np.linalg.norm(dx[b]) + np.linalg.norm(r[b]))
    if bad is not None:
        assert np.all(dx[1] == 0.0)
