"""One-electron integrals at the edges of the wave's work split.

A wave takes 64 primitive pairs at a time and deals (primitive pair, nucleus)
items to 64 lanes: contractions past one chunk (12 x 12 = 144 pairs), one, 63,
64, 65 and 130 nuclei, every class of s, p and d shells, centres without
charge.  Tolerance: sums of up to 144 x 130 terms of one sign in 64 bits, so
1e-12 of the largest element.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _even(base, n, ratio):
    return tuple(base * ratio ** k for k in range(n))


def _lattice(n, seed):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    return g * 3.1 + rng.uniform(-0.4, 0.4, (n, 3))


def _molecule(kind, natom):
    rng = np.random.default_rng(natom)
    if kind == "contracted":
        c = lambda n: tuple(rng.uniform(0.1, 1.0, n))  # noqa: E731
        basis = {8: [(0, _even(0.07, 12, 2.6), c(12)), (1, _even(0.1, 9, 2.5), c(9)), (2, (0.9,), (1.0,))],
                 2: [(2, _even(0.3, 12, 2.0), c(12)), (1, (0.4,), (1.0,)), (0, (0.2,), (1.0,))]}
        Z = [8 if a % 2 == 0 else 2 for a in range(natom)]
    else:
        basis = {z: [(0, (0.5, 3.0), (0.6, 0.5))] for z in (0, 2, 8)}
        basis[8] = [(2, (0.8,), (1.0,)), (0, (1.1,), (1.0,))]
        Z = [8 if a == 0 else 0 if a % 5 == 1 else 2 for a in range(natom)]
    return W.attach_basis(Z, _lattice(natom, natom), basis)


@pytest.mark.parametrize("kind,natom", [("contracted", 1), ("contracted", 3), ("many", 63), ("many", 64),
                                        ("many", 65), ("many", 130)])
def test_against_oracle(kind, natom):
    import oracle
    from paper_1708_00033_amd import hfx
    m = _molecule(kind, natom)
    S, H, _ = hfx.Context().load(m).core()
    So, To, Vo, _ = oracle.Basis(m).one_electron()
    Ho = To + Vo
    assert np.abs(S - So).max() <= 1e-12 * np.abs(So).max()
    assert np.abs(H - Ho).max() <= 1e-12 * np.abs(Ho).max()
    assert np.array_equal(S, S.T) and np.array_equal(H, H.T)


def test_centre_without_charge_far_away():
    from paper_1708_00033_amd import hfx
    import oracle
    m = W.attach_basis([2, 0], np.array([[0.0, 0.0, 0.0], [1e200, 0.0, 0.0]]), {2: [(0, (0.5, 3.0), (0.6, 0.5))], 0: []})
    S, H, _ = hfx.Context().load(m).core()
    ref = oracle.Basis(W.attach_basis([2], np.zeros((1, 3)), {2: [(0, (0.5, 3.0), (0.6, 0.5))]})).one_electron()
    assert np.abs(S - ref[0]).max() <= 1e-12 and np.abs(H - ref[1] - ref[2]).max() <= 1e-12 * np.abs(H).max()
