"""What the two kinds of kernel timing time: every plan by itself, or the
launches of a build, where the plans of a class are joined."""
from __future__ import annotations

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", [0, 1, 3])
@pytest.mark.parametrize("mixed", [False, True])
def test_plans_and_launches(form, mixed):
    import torch
    from paper_1708_00033_amd import hfx
    m = W.water_cluster(5, 3)
    ctx = hfx.Context(precision=hfx.HFX_PREC_MIXED if mixed else hfx.HFX_PREC_FP64)
    ctx.set_class_tuning(-1, 0, -1, form, -1)
    ctx.load(m)
    D = torch.tensor(W.random_orthonormal_density(m.nbf, m.nocc, 8), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    ref, F = torch.empty_like(D), torch.empty_like(D)
    ctx.build_fock_dev(D.data_ptr(), ref.data_ptr(), s)
    torch.cuda.synchronize()
    for mode in (hfx.HFX_TIME_PLANS, hfx.HFX_TIME_LAUNCHES, hfx.HFX_TIME_PLANS):
        ctx.kernel_timing(mode)
        for _ in range(3):
            ctx.build_fock_dev(D.data_ptr(), F.data_ptr(), s)
        torch.cuda.synchronize()
        assert (F - ref).abs().max().item() <= 1e-13 * ref.abs().max().item()   # order of sums
        ms, n = ctx.kernel_times()
        plans = ctx.plans()
        for k in range(21):
            own = [p for p in plans if p["cls"] == k]
            assert n[k] == 3 and ms[k] > 0
            timed = [p for p in own if p["launches"]]
            assert all(p["launches"] == 3 for p in timed)
            # register-tiled plans (ket primitive counts 1, 3, 9) have kernels of their own
            apart = [p for p in own if p["persistent"] in (3, 4)]
            rest = len(own) - len(apart)
            want = len(own) if mode == hfx.HFX_TIME_PLANS else len(apart) + (rest > 0)
            assert len(timed) == want, (hfx.CLASS_NAMES[k], mode)
            assert sum(p["ms"] for p in own) == pytest.approx(ms[k])
    ctx.kernel_timing(False)
    ctx.build_fock_dev(D.data_ptr(), F.data_ptr(), s)
    torch.cuda.synchronize()
    assert (ctx.kernel_times()[1] == 0).all()
