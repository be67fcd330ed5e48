"""Parameters and gradients back on the host: through pinned memory up to 32 MiB
of them, an array at a time above, and nothing large kept in host memory."""
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


# padded words below, at and above 8,388,608: 64 x 129,024 + 129,024, one more
# panel of 64 rows, and several layers of odd widths
@pytest.mark.parametrize("dims", [(5, 70, 3), (64, 129_024), (64, 129_088), (33, 3001, 2900, 7)])
def test_round_trip(ctx, dims):
    import torch
    mlp = nnc.nnc_train_create(ctx.h, list(dims), 4, nnc.PREC_CODES["fp32"], 1)
    n = nnc.nnc_train_num_params(ctx.h, mlp)
    p = np.arange(n, dtype=np.float64) % 8191 / 64.0 - 60.0  # FP32 numbers
    nnc.nnc_train_set_params(ctx.h, mlp, p)
    assert np.array_equal(nnc.nnc_train_get_params(ctx.h, mlp), p)
    small = 1e-3 * p
    nnc.nnc_train_set_params(ctx.h, mlp, small)
    X, Y = (torch.ones((4, d), dtype=torch.float64, device="cuda") for d in (dims[0], dims[-1]))
    nnc.nnc_train_step(ctx.h, mlp, X.data_ptr(), Y.data_ptr(), 1e-3)
    g = nnc.nnc_train_get_grads(ctx.h, mlp)
    nnc.nnc_train_destroy(ctx.h, mlp)
    assert g.shape == (n,) and np.all(np.isfinite(g))
    # inputs of one: every row of dW_1 repeats db_1
    k = dims[1] * dims[0]
    assert np.allclose(g[:k].reshape(dims[1], dims[0]), g[k:k + dims[1], None], rtol=1e-5, atol=1e-30)


def mapped():
    """Bytes of device and pinned host memory that this process has mapped."""
    total = 0
    with open("/proc/self/maps") as f:
        for line in f:
            part = line.split()
            if len(part) > 5 and "/dev/dri/render" in part[5]:
                lo, hi = part[0].split("-")
                total += int(hi, 16) - int(lo, 16)
    return total


def test_large_trainer_keeps_no_host_copy(ctx):
    import torch
    host, free = mapped(), torch.cuda.mem_get_info()[0]
    mlp = nnc.nnc_train_create(ctx.h, [64, 600_000], 4, nnc.PREC_CODES["bf16"], 1)  # 156 MB of parameters
    pinned = mapped() - host - (free - torch.cuda.mem_get_info()[0])
    nnc.nnc_train_destroy(ctx.h, mlp)
    assert pinned < 100 << 20, pinned
