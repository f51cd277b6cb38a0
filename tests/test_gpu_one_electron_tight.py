"""S and H of tight functions far from the origin, and of diffuse ones.

The product of two Gaussians lies between their centres; its distance to either
has to keep the digits that a function of width 1e-3 at coordinates of some bohr
needs.  Against the oracle (McMurchie-Davidson, distances from A - B).
Tolerance: an element of S is a sum of up to nine primitive products of three
one-dimensional overlaps of at most six steps, some 100 roundings of 1.1e-16;
H the same against its largest element.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

EXPS = ((1e6, 3e4, 900.0), (2e5,), (40.0, 2.0), (0.2,))


@pytest.mark.parametrize("shift", [0.0, 7.3, 50.7])
@pytest.mark.parametrize("far", [0.0, 0.4, 3.1])
def test_tight_functions(shift, far):
    import oracle
    from paper_1708_00033_amd import hfx
    xyz = np.array([[0.1, -0.2, 0.3], [0.1 + 0.48 * far, -0.2 + 0.6 * far, 0.3 - 0.64 * far]]) + shift
    shells = [W.Shell(a, l, np.array(e), np.linspace(0.7, 0.4, len(e))) for a in (0, 1) for l in (0, 1, 2) for e in EXPS]
    m = W.Molecule(np.array([2, 2 if far else 0], dtype=np.int32), xyz, shells)
    S, T, V, _ = oracle.Basis(m).one_electron()
    Sg, Hg, _ = hfx.Context().load(m).core()
    es, eh = float(np.abs(Sg - S).max()), float(np.abs(Hg - (T + V)).max() / np.abs(T + V).max())
    print(f"S {es:.1e} H {eh:.1e}")
    assert es <= 1.1e-14
    assert eh <= 1.1e-14
    assert np.array_equal(Sg, Sg.T) and np.array_equal(Hg, Hg.T)
