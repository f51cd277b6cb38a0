"""Passes of one network on several streams: the second must not depend on
hidden work of the first.

New parameters are set, a first forward is queued on a stream that is still
busy with other work, and a second one on an idle stream runs meanwhile.  Both
give what a single stream gives, bit for bit (the same kernels on the same
weights).
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import guess as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("update", ["set", "adam"])
def test_second_stream_sees_new_weights(update):
    import torch
    from paper_1708_00033_amd import hfx
    rng = np.random.default_rng(4)
    counts = (40, 70, 30)
    X = torch.tensor(rng.normal(size=(sum(counts), G.NFEAT)).astype(np.float32), device="cuda")
    n = sum(c * k for c, k in zip(counts, G.HEAD_OUT))
    T = torch.tensor(rng.normal(size=n).astype(np.float32) * 0.03, device="cuda")

    def params(seed):
        p = G.init_params(seed, fmean=np.zeros(G.NFEAT), fscale=np.ones(G.NFEAT), tscale=np.full(3, 0.05))
        for t, k in enumerate(G.HEAD_OUT):
            p[f"H{t}"] = np.random.default_rng(seed + t).normal(size=(k, G.HIDDEN)) * 0.05
        return G.pack(p).astype(np.float32)

    net = hfx.GuessNet(0, params(1))
    old, ref, a, b = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(4))
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    net.forward_dev(X.data_ptr(), counts, old.data_ptr(), sb.cuda_stream)
    net.grad_dev(X.data_ptr(), counts, T.data_ptr(), sb.cuda_stream)
    busy = torch.rand(8192, 8192, device="cuda")
    out = torch.empty_like(busy)
    torch.cuda.synchronize()
    if update == "set":
        net.set_params(params(2))
    else:
        net.adam(1e-2, sb.cuda_stream)
    torch.cuda.synchronize()
    with torch.cuda.stream(sa):
        for _ in range(20):
            torch.mm(busy, busy, out=out)
    net.forward_dev(X.data_ptr(), counts, a.data_ptr(), sa.cuda_stream)
    net.forward_dev(X.data_ptr(), counts, b.data_ptr(), sb.cuda_stream)
    torch.cuda.synchronize()
    net.forward_dev(X.data_ptr(), counts, ref.data_ptr(), sb.cuda_stream)
    torch.cuda.synchronize()
    assert not torch.equal(ref, old)
    assert torch.equal(a, ref) and torch.equal(b, ref)
