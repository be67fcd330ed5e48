"""A network whose packed operands fit in device memory but not what has to stand
beside them is created on row-major operands, as it was without packed ones."""
import numpy as np
import pytest

from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu


def fill(room):
    """All device memory but about `room` bytes."""
    import torch
    held = []
    while torch.cuda.mem_get_info()[0] - room > 64 << 20:
        held.append(torch.empty(torch.cuda.mem_get_info()[0] - room - (32 << 20), dtype=torch.uint8, device="cuda"))
    return held


# created with the layer sum (many hidden units against inputs), and with
# forward-over-reverse and then changed to it
@pytest.mark.parametrize("dims,points,method", [((100, 1000, 1024, 1000, 3), 1000, "layersum"),
                                                ((2000, 60, 1000, 3), 100, "for")])
def test_less_memory_than_packed_operands_need(dims, points, method):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    acts = ["tanh"] * (len(dims) - 2) + ["identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=21, bias_scale=0.2)
    ctx = nnc.Context(0)
    X, Lam = (torch.as_tensor(v, device="cuda") for v in datagen.points(dims[0], dims[-1], points, seed=22))

    def hessians(net):
        H = net.eval_hess_lag(X, Lam)[[0, points // 2, points - 1]].cpu().numpy()
        torch.cuda.empty_cache()
        return H

    def free():
        return torch.cuda.mem_get_info()[0]

    want = torch.empty((points, dims[0], dims[0]), dtype=torch.float64, device="cuda")  # room for the results later
    at = free()
    net = ctx.net(dims, acts, Ws, bs, prec="fp32", max_points=points)  # with all the memory there is
    assert net.hess_method == method
    created = at - free()
    net.set_hess_method("layersum")
    packed = at - free()
    ref = hessians(net)
    net.destroy()
    # beyond row-major operands: half as much again for P and U, and the packed weights
    dp = [(d + 63) // 64 * 64 for d in dims[1:-1]]
    more = points * dims[0] * 2 * (sum(dp) + sum(dp[:-1])) + 6 * sum(a * b for a, b in zip(dp, dp[1:]))
    hog = []
    try:
        if method == "for":
            net = ctx.net(dims, acts, Ws, bs, prec="fp32", max_points=points)
        hog = fill(packed - more // 2 - (created if method == "for" else 0))
        if method == "layersum":
            net = ctx.net(dims, acts, Ws, bs, prec="fp32", max_points=points)
        net.set_hess_method("layersum")
        del want
        torch.cuda.empty_cache()
        got = hessians(net)
        net.destroy()
    finally:
        del hog
        torch.cuda.empty_cache()
        ctx.close()
    for h, r in zip(got, ref):
        assert np.linalg.norm(h - r) < 1e-5 * np.linalg.norm(r)
