"""One launch for all ket lists of a class against one launch per list.

Builds whose launches are timed keep a launch per plan; the others join the
plans of a class.  Both are held to the oracle in every launch form (one task
per workgroup, persistent, one task per wave, register-tiled, where plans stay
apart), both precisions, for a molecule and a ragged batch.  Tolerance: FP64
sums of some 10^4 terms, 1e-12 of the largest element; FP32 quartets below
1e-6 of it, 1e-7 each.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1, 2, 3])
@pytest.mark.parametrize("mixed", [False, True])
def test_joined_and_single_launches(form, mixed):
    import oracle
    import torch
    from paper_1708_00033_amd import hfx
    mols = [W.water_cluster(3, 7), W.water_dimer(1, W.BASIS_SPD)]
    ref, dens = [], []
    for i, m in enumerate(mols):
        B = oracle.Basis(m)
        D = W.random_symmetric(m.nbf, 11 + i, 0.2)
        _, T, V, _ = B.one_electron()
        J, K, _ = B.jk(D, 1e-10)
        ref.append((T + V + 2 * J - K).ravel())
        dens.append(D.ravel())
    ref = np.concatenate(ref)
    ctx = hfx.Context(precision=hfx.HFX_PREC_MIXED if mixed else hfx.HFX_PREC_FP64)
    ctx.set_class_tuning(-1, 512, -1, form, -1)
    ctx.load_batch(mols)
    assert any(sum(q["cls"] == p["cls"] for q in ctx.plans()) > 1 for p in ctx.plans())
    D = torch.tensor(np.concatenate(dens), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    tol = (1e-9 if mixed else 1e-12) * np.abs(ref).max()
    for timing in (False, True, False):
        ctx.kernel_timing(timing)
        F = torch.full_like(D, float("nan"))
        ctx.build_fock_dev(D.data_ptr(), F.data_ptr(), s)
        torch.cuda.synchronize()
        assert np.abs(F.cpu().numpy() - ref).max() <= tol, timing
