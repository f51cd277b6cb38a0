"""max|D| of a mixed build: where the largest element lies, and what finding it costs."""
from __future__ import annotations

import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _batch(n_small):
    return [W.h2(1.4) for _ in range(n_small // 2)] + [W.water_cluster(16, 5)] + \
           [W.h2(1.4) for _ in range(n_small - n_small // 2)]


def test_largest_element_anywhere():
    """The FP32 share of the quartets depends on max|D| only: the same for one
    large element, of either sign, at any place of any molecule."""
    import torch
    from paper_1708_00033_amd import hfx
    mols = _batch(6)
    ctx = hfx.Context(precision=hfx.HFX_PREC_MIXED).load_batch(mols)
    nbf, _, off, tot = ctx.layout
    s = torch.cuda.current_stream().cuda_stream
    rng = np.random.default_rng(1)
    base = rng.uniform(-1e-3, 1e-3, size=tot)
    F = torch.empty(tot, dtype=torch.float64, device="cuda")

    def fp32(D):
        return ctx.build_fock_dev(torch.tensor(D, device="cuda").data_ptr(), F.data_ptr(), s, stats=True).quartets_fp32

    few, big = None, int(off[3])
    none = fp32(base)
    for i in (0, 1, 3, big, big + 63, big + 64, big + 255, big + 256, big + int(nbf[3]) ** 2 - 1, tot - 1):
        for v in (3.0, -3.0):
            D = base.copy()
            D[i] = v
            got = fp32(D)
            few = got if few is None else few
            assert got == few < none, (i, v)


def test_cost_on_a_ragged_batch():
    """Three thousand small molecules beside a large one: a mixed build whose
    classes all stay in FP64 differs from an FP64 build by max|D| alone, which
    may not take as long as the build."""
    import torch
    from paper_1708_00033_amd import hfx
    ctx = hfx.Context().load_batch(_batch(3000))
    D = torch.tensor(np.random.default_rng(2).uniform(-1, 1, size=ctx.layout[3]), device="cuda")
    F = torch.empty_like(D)
    s = torch.cuda.current_stream().cuda_stream

    def ms():
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ctx.build_fock_dev(D.data_ptr(), F.data_ptr(), s)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best * 1e3

    fp64 = ms()
    ctx.configure(precision=hfx.HFX_PREC_MIXED)
    ctx.set_class_precision(-1, 0)
    mixed = ms()
    print(f"FP64 {fp64:.2f} ms, mixed without FP32 classes {mixed:.2f} ms")
    assert mixed < 2 * fp64
