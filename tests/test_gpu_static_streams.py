"""nnc_eval_g_static beside other calls on the same network, queued on another
stream: it writes nothing that they use, nor they what it uses."""
import numpy as np
import pytest

from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp64"])
@pytest.mark.parametrize("B", [1, 21, 40])
def test_static_call_beside_others(prec, B):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    ctx = nnc.Context(0)
    dims = (200, 2000, 2048, 1500, 3)  # wide enough for rows staged in K slices
    acts = ["tanh", "tanh", "tanh", "identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=41, bias_scale=0.2)
    X, _ = datagen.points(dims[0], dims[-1], 2 * B, seed=42)
    net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=B)
    x0, x1 = (torch.as_tensor(X[k * B:(k + 1) * B], device="cuda").contiguous() for k in (0, 1))
    J0, g0, g1 = net.eval_jac_g(x0).clone(), net.eval_g(x0).clone(), net.eval_g(x1).clone()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    J = [torch.empty_like(J0) for _ in range(20)]
    g = [torch.empty_like(g0) for _ in range(20)]
    s = [torch.empty_like(g1) for _ in range(60)]
    torch.cuda.synchronize()
    try:
        for k in range(20):
            assert nnc.nnc_set_stream(ctx.h, one.cuda_stream) == nnc.NNC_OK
            assert nnc.nnc_eval_jac_g(ctx.h, net.h, B, x0.data_ptr(), J[k].data_ptr()) == nnc.NNC_OK
            assert nnc.nnc_eval_g(ctx.h, net.h, B, x0.data_ptr(), None, g[k].data_ptr()) == nnc.NNC_OK
            assert nnc.nnc_set_stream(ctx.h, two.cuda_stream) == nnc.NNC_OK
            for i in range(3):
                out = s[3 * k + i]
                assert nnc.nnc_eval_g_static(ctx.h, net.h, B, x1.data_ptr(), None, out.data_ptr()) == nnc.NNC_OK
        torch.cuda.synchronize()
    finally:
        nnc.nnc_set_stream(ctx.h, None)
    assert all(torch.equal(t, J0) for t in J)
    assert all(torch.equal(t, g0) for t in g)
    assert all(torch.equal(t, g1) for t in s)
    net.destroy()
    ctx.close()
