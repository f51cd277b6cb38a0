"""GPU parity of the cooperative Rys kernels where they can go wrong: contracted
d and p shells (several bra and ket primitives per step), arguments of the
quadrature from 0 to far above its table (T >= 60), batches with one ket and
with a remainder, every launch form, digestion, precision and density count."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

# the classes of the cooperative kernels hold 18-36 bra components; the FP64
# bound is the one of the other parity tests (1e-10 on F), the FP32 bound that
# of test_gpu_fp32_full (2e-5 relative)
TOL64, RTOL32 = 1e-10, 2e-5


def _chain(natom):
    """natom centres at 0, 0.9, 7 and 30 bohr with contracted and single p and
    d shells: rho R^2 from 0 to several hundred."""
    basis = {8: [(0, (1.3, 0.4), (0.6, 0.5)), (1, (1.1, 0.35), (0.5, 0.6)), (1, (0.2,), (1.0,)),
                 (2, (1.7, 0.6), (0.4, 0.7)), (2, (0.45,), (1.0,))]}
    xyz = np.array([[0.0, 0.0, 0.0], [0.5, -0.6, 0.45], [3.1, 5.2, -3.4], [-17.0, 19.0, 16.0]])[:natom]
    return W.attach_basis([8] * natom, xyz, basis)


def _hfx():
    from paper_1708_00033_amd import hfx
    return hfx


@pytest.mark.parametrize("natom", [1, 2, 4])
def test_contracted_shells_all_arguments(natom):
    import oracle
    hfx = _hfx()
    m = _chain(natom)
    B = oracle.Basis(m)
    D = W.random_symmetric(m.nbf, 5, 0.1)
    J, K, _ = B.jk(D, 0.0)
    S, T, V, _ = B.one_electron()
    ref = T + V + 2 * J - K
    for digest in (hfx.HFX_DIGEST_LDS, hfx.HFX_DIGEST_GLOBAL, hfx.HFX_DIGEST_PRIVATE):
        for form in (0, 1, 2):
            ctx = hfx.Context(schwarz_tau=0.0, digest=digest).load(m)
            ctx.set_class_tuning(-1, 256, 0, form)
            F, _ = ctx.build_fock(D)
            assert np.abs(F - ref).max() < TOL64, (digest, form)
    ctx = hfx.Context(schwarz_tau=0.0).load(m)
    assert np.abs(ctx.schwarz() - B.schwarz()).max() < 1e-12
    mx = hfx.Context(schwarz_tau=0.0, precision=hfx.HFX_PREC_MIXED, fp32_tau=1e300).load(m)
    F, st = mx.build_fock(D)
    assert st.quartets_fp32 > 0
    assert np.abs(F - ref).max() <= RTOL32 * np.abs(2 * J - K).max()


@pytest.mark.parametrize("ndens", [1, 3, 9])
def test_several_densities(ndens):
    """Small sums per density in LDS, densities in groups that fit."""
    import oracle
    import torch
    hfx = _hfx()
    m = _chain(3)
    B = oracle.Basis(m)
    D = np.stack([W.random_symmetric(m.nbf, 20 + d, 0.1) for d in range(ndens)])
    dD = torch.tensor(D, device="cuda")
    for digest in (hfx.HFX_DIGEST_LDS, hfx.HFX_DIGEST_GLOBAL):
        ctx = hfx.Context(digest=digest).load(m)
        dJ, dK = torch.empty_like(dD), torch.empty_like(dD)
        ctx.build_jk_multi_dev(ndens, dD.data_ptr(), dJ.data_ptr(), dK.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        for d in range(ndens):
            J, K, _ = B.jk(D[d], 1e-10)
            assert np.abs(dJ[d].cpu().numpy() - J).max() < TOL64
            assert np.abs(dK[d].cpu().numpy() - K).max() < TOL64
