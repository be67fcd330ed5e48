"""nnc_autotune of a layer-sum network tunes what the network runs: each packed
sweep product has a row in the table afterwards, results stay right, a context
that reads the file back takes the same choices, and so do other networks of the
context with products of the same shape."""
import json

import numpy as np
import pytest

from oracle import nn as O
from paper_2509_22462_amd import datagen, nnc

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-5, "bf16": 2e-2, "fp64": 1e-10}


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp64"])
@pytest.mark.parametrize("dims,B", [((37, 150, 70, 90, 5), 3), ((90, 300, 1500, 4), 1)])
def test_packed_products_are_tuned(tmp_path, monkeypatch, prec, dims, B):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("NNC_AUTOTUNE_CACHE", str(cache))
    code = nnc.PREC_CODES[prec]
    acts = ["tanh"] * (len(dims) - 2) + ["identity"]
    Ws, bs = datagen.mlp_weights(dims, seed=61, bias_scale=0.2)
    X, Lam = datagen.points(dims[0], dims[-1], B, seed=62)
    pad = [(d + 63) // 64 * 64 for d in dims[1:-1]]
    shapes = [(B * dims[0], b, a) for a, b in zip(pad, pad[1:])]

    def check(ctx, net):
        H = net.eval_hess_lag(X, Lam).cpu().numpy()
        for b in range(B):
            R = O.hess_layersum(Ws, bs, acts, X[b], Lam[b])
            assert np.linalg.norm(H[b] - R) < TOL[prec] * np.linalg.norm(R)
        return H, [nnc.nnc_autotune_query(ctx.h, code, *s, 0, 0) for s in shapes]

    ctx = nnc.Context(0)
    net, other = (ctx.net(dims, acts, Ws, bs, prec=prec, max_points=most, hess="layersum") for most in (B, 4 * B))
    assert check(ctx, net)[1] == [-1] * len(shapes)
    assert nnc.nnc_autotune(ctx.h, net.h, B) == nnc.NNC_OK, nnc.nnc_last_error(ctx.h)
    H, rows = check(ctx, net)
    assert min(rows) >= 0
    assert np.array_equal(check(ctx, other)[0], H)
    ctx.close()
    lines = [json.loads(t) for t in cache.read_text().splitlines()]
    assert sorted((r["M"], r["N"], r["K"]) for r in lines if r["splits"] == 0) == sorted(set(shapes))
    assert all(r["validated"] and r["rejected"] == 0 and r["max_rel_err"] <= TOL[prec] for r in lines)
    ctx = nnc.Context(0)
    net = ctx.net(dims, acts, Ws, bs, prec=prec, max_points=B, hess="layersum")
    again, read = check(ctx, net)
    assert read == rows and np.array_equal(again, H)
    ctx.close()
