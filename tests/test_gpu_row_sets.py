"""Rows of W in LDS at every size: no class of d-d or d-p bras is left to global
updates, between whole rows and windows either.

Sizes around the largest whole rows of each bra class and table, up to the first
windows.  Plans: one centre with s, p and d shells and far d and s shells that
make up the number of functions.  J and K: 66 waters and seven far s functions
(1261), in the range where the d-d classes with the largest tables take windows
and the others whole rows, against the global-atomic digestion, 1e-12 of the
largest element as between summation orders elsewhere.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ONE = np.array([1.0])


def _sized(n):
    """n functions: s, p and d shells on one centre, the rest far away."""
    near = [W.Shell(0, l, ONE * e, ONE) for l in (0, 1, 2) for e in (0.4, 1.1)]
    k, s = divmod(n - 20, 6)
    far = [W.Shell(1 + i, 2, ONE * 0.8, ONE) for i in range(k)] + [W.Shell(1 + k + i, 0, ONE * 0.8, ONE) for i in range(s)]
    xyz = np.concatenate([np.zeros((1, 3)), 200.0 + 100.0 * np.array([(i % 8, i // 8 % 8, i // 64) for i in range(k + s)])])
    m = W.Molecule(np.array([2] + [0] * (k + s), dtype=np.int32), xyz, near + far)
    assert m.nbf == n
    return m


def test_every_size_keeps_lds_rows():
    from paper_1708_00033_amd import hfx
    ctx = hfx.Context()
    for n in list(range(1196, 1300, 3)) + list(range(1300, 1900, 12)) + [2040, 2100, 3000]:
        ctx.load(_sized(n))
        for p in ctx.plans():
            if hfx.CLASS_NAMES[p["cls"]][:3] in ("(dp", "(dd"):
                assert p["mode"] in (hfx.HFX_DIGEST_LDS, hfx.HFX_DIGEST_LDS_D), (n, hfx.CLASS_NAMES[p["cls"]])


@pytest.mark.parametrize("form", [0, 1])
def test_whole_rows_and_windows_of_one_bra_class(form):
    import torch
    from paper_1708_00033_amd import hfx
    m = W.water_cluster(66, 1)
    far = m.natom
    m = W.Molecule(np.append(m.Z, np.int32(0)), np.concatenate([m.xyz, [[300.0, 0.0, 0.0]]]),
                   m.shells + [W.Shell(far, 0, ONE * (0.5 + 0.1 * i), ONE) for i in range(7)])
    assert m.nbf == 1261
    D = torch.tensor(W.random_orthonormal_density(m.nbf, m.nocc, 5), device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    ctx = hfx.Context().load(m)
    ref, out = torch.empty_like(D), torch.empty_like(D)
    for cj, ck in ((1.0, 0.0), (0.0, -1.0)):
        ctx.set_class_tuning(-1, 0, -1, 0, 1)
        ctx.build_2e_dev(D.data_ptr(), cj, ck, ref.data_ptr(), s)
        ctx.set_class_tuning(-1, 0, -1, form, -1)
        st = ctx.build_2e_dev(D.data_ptr(), cj, ck, out.data_ptr(), s, stats=True)
        assert st.quartets_fp64 == int(ctx.class_counts()[:, 0].sum())
        assert (out - ref).abs().max().item() <= 1e-12 * ref.abs().max().item(), (cj, ck)
