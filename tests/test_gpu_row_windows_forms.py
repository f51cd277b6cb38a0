"""Column windows of W in every launch form, precision and number of densities.

Eight waters whose atoms are listed four before and four after far d shells, so
that their functions lie at both ends of 1330 functions (d-d bras windowed),
1900 (d-p bras too) and 2400 (whole rows or windows by ket class) and their
pairs in windows that differ.  Every class keeps its rows in LDS.  With a
density on the waters alone, their blocks of J and K are those of the waters
loaded without the far shells, by global atomics; 1e-12 of the largest element
as between summation orders elsewhere; mixed builds: FP32 quartets below 1e-6
of it, 1e-7 each.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _split_waters(n):
    """The waters with n functions in all, and without the far shells; the waters' functions among n."""
    w = W.water_cluster(8, 21)
    half = w.natom // 2
    k, s = divmod(n - w.nbf, 6)
    far_xyz = 300.0 + 100.0 * np.array([(i % 8, i // 8 % 8, i // 64) for i in range(k + s)])
    shells = [x for x in w.shells if x.atom < half]
    n0 = sum(x.nbf for x in shells)
    shells += [W.Shell(half + i, 2 if i < k else 0, np.array([0.8]), np.array([1.0])) for i in range(k + s)]
    shells += [W.Shell(x.atom + k + s, x.l, x.exps, x.coefs) for x in w.shells if x.atom >= half]
    m = W.Molecule(np.concatenate([w.Z[:half], np.zeros(k + s, dtype=np.int32), w.Z[half:]]).astype(np.int32),
                   np.concatenate([w.xyz[:half], far_xyz, w.xyz[half:]]), shells)
    assert m.nbf == n
    import torch
    at = np.concatenate([np.arange(n0), np.arange(n - (w.nbf - n0), n)])
    return m, w, torch.tensor(at, device="cuda")


def _reference(w, D):
    import torch
    from paper_1708_00033_amd import hfx
    s = torch.cuda.current_stream().cuda_stream
    ctx = hfx.Context(digest=hfx.HFX_DIGEST_GLOBAL).load(w)
    out = []
    for cj, ck in ((1.0, 0.0), (0.0, -1.0)):
        G = torch.empty_like(D)
        ctx.build_2e_dev(D.data_ptr(), cj, ck, G.data_ptr(), s)
        out.append(G)
    torch.cuda.synchronize()
    return out


def _put(D, at, n):
    import torch
    big = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    big[at[:, None], at] = D
    return big


@pytest.mark.parametrize("n", [1330, 1900, 2400])
def test_one_density(n):
    import torch
    from paper_1708_00033_amd import hfx
    m, w, at = _split_waters(n)
    s = torch.cuda.current_stream().cuda_stream
    D = torch.tensor(W.random_symmetric(w.nbf, 3, 0.2), device="cuda")
    ref = _reference(w, D)
    big = _put(D, at, n)
    G = torch.empty_like(big)
    ctx = hfx.Context().load(m)
    for mixed in (False, True):
        ctx.configure(precision=hfx.HFX_PREC_MIXED if mixed else hfx.HFX_PREC_FP64)
        tol = 1e-9 if mixed else 1e-12
        for form in (0, 1, 2, 3, 4):
            ctx.set_class_tuning(-1, 0, -1, form, -1)
            for p in ctx.plans():
                assert p["mode"] in (hfx.HFX_DIGEST_LDS, hfx.HFX_DIGEST_LDS_D), (form, p)
            for (cj, ck), r in zip(((1.0, 0.0), (0.0, -1.0)), ref):
                ctx.build_2e_dev(big.data_ptr(), cj, ck, G.data_ptr(), s)
                torch.cuda.synchronize()
                d = (G[at[:, None], at] - r).abs().max().item()
                assert d <= tol * r.abs().max().item(), (mixed, form, cj, ck)


@pytest.mark.parametrize("n", [1330, 1900, 2400])
@pytest.mark.parametrize("ndens", [2, 5])
def test_several_densities(n, ndens):
    import torch
    from paper_1708_00033_amd import hfx
    m, w, at = _split_waters(n)
    s = torch.cuda.current_stream().cuda_stream
    Ds = [torch.tensor(W.random_symmetric(w.nbf, 30 + d, 0.2), device="cuda") for d in range(ndens)]
    big = torch.stack([_put(D, at, n) for D in Ds])
    J, K = torch.empty_like(big), torch.empty_like(big)
    for digest in (hfx.HFX_DIGEST_LDS_D, hfx.HFX_DIGEST_GLOBAL):
        ctx = hfx.Context(digest=digest).load(m)
        ctx.build_jk_multi_dev(ndens, big.data_ptr(), J.data_ptr(), K.data_ptr(), s)
        torch.cuda.synchronize()
        for d, D in enumerate(Ds):
            rj, rk = _reference(w, D)
            assert (J[d][at[:, None], at] - rj).abs().max().item() <= 1e-12 * rj.abs().max().item(), (digest, d)
            assert (K[d][at[:, None], at] - rk).abs().max().item() <= 1e-12 * rk.abs().max().item(), (digest, d)
