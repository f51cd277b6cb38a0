"""The guess network's row-block kernels at the edges of their blocks.

Rows are walked in blocks of 32 of one pair type and the weight gradients in
chunks of 32 blocks: types without rows, one row, full and just overfull
blocks, and more than one chunk with types that begin inside one.
Tolerances: two BF16 operands of relative error 2^-9 per product, over four
layers forward and four back, stay below 2e-2 of an array's norm; the bias sums
and the loss are held to the same.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import guess as G

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.ravel(a) - np.ravel(b)) / max(np.linalg.norm(np.ravel(b)), 1e-30)


@pytest.mark.parametrize("counts", [(1, 0, 0), (0, 0, 1), (0, 33, 0), (31, 32, 33), (64, 1, 65), (40, 1100, 1000)])
def test_row_blocks_and_chunks(counts):
    import torch
    from paper_1708_00033_amd import hfx
    rng = np.random.default_rng(sum(counts))
    M = sum(counts)
    X = rng.normal(size=(M, G.NFEAT)).astype(np.float32)
    p = G.init_params(3, fmean=rng.normal(size=G.NFEAT) * 0.1, fscale=np.full(G.NFEAT, 1.3),
                      tscale=np.array([0.05, 0.03, 0.02]))
    for t, n in enumerate(G.HEAD_OUT):
        p[f"H{t}"] = rng.normal(size=(n, G.HIDDEN)) * 0.05
        p[f"c{t}"] = rng.normal(size=n) * 0.01
    flat = G.pack(p).astype(np.float32)
    p = G.unpack(flat.astype(np.float64))
    T = [(rng.normal(size=(c, n)) * 0.03).astype(np.float32) for c, n in zip(counts, G.HEAD_OUT)]
    net = hfx.GuessNet(0, flat)
    dX = torch.tensor(X, device="cuda")
    dT = torch.tensor(np.concatenate([x.ravel() for x in T]), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    out = torch.full((dT.numel() + 64,), 7.0, dtype=torch.float32, device="cuda")
    net.forward_dev(dX.data_ptr(), counts, out.data_ptr(), s)
    torch.cuda.synchronize()
    Y = out.cpu().numpy()
    assert (Y[dT.numel():] == 7.0).all()
    o = 0
    for c, n, ref in zip(counts, G.HEAD_OUT, G.predict_blocks(p, X.astype(np.float64), counts)):
        if c:
            assert _rel(Y[o:o + c * n], np.asarray(ref).ravel()) < 2e-2
        o += c * n
    lo, go = G.loss_and_grad(p, X.astype(np.float64), counts, [x.astype(np.float64) for x in T])
    got = []
    for _ in range(2):   # the second pass finds the scratch of the first
        loss = net.grad_dev(dX.data_ptr(), counts, dT.data_ptr(), s)
        assert abs(loss - lo) <= 2e-2 * lo
        got.append(net.get_grads())
        gr = G.unpack(got[-1].astype(np.float64))
        for name, _ in G.param_shapes()[:G.TRAINABLE]:
            assert _rel(gr[name], go[name]) < 2e-2, name
        for name, _ in G.param_shapes()[G.TRAINABLE:]:
            assert not gr[name].any()
    assert np.array_equal(got[0], got[1])
