"""Schwarz bounds of more pairs than one launch takes.

The d-p and d-d bounds take a workgroup per pair and launches of at most 2^20
workgroups.  1450 equal d shells and 725 equal p shells on one centre have
1,051,975 d-d and 1,051,250 d-p pairs; every one of a kind has the bound of the
same pair in a small molecule, by the same arithmetic, so to the last bit.  The
threshold leaves no pair, so that nothing is planned.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _shells(nd, n_p):
    d = [W.Shell(0, 2, np.array([0.7, 0.3]), np.array([0.6, 0.5])) for _ in range(nd)]
    p = [W.Shell(0, 1, np.array([0.4]), np.array([1.0])) for _ in range(n_p)]
    return W.Molecule(np.array([2], dtype=np.int32), np.zeros((1, 3)), d + p)


def test_bounds_beyond_one_launch():
    from paper_1708_00033_amd import hfx
    nd, n_p = 1450, 725
    assert nd * (nd + 1) // 2 > 1 << 20 and nd * n_p > 1 << 20
    small = hfx.Context(schwarz_tau=1e6).load(_shells(2, 2)).schwarz()
    Q = hfx.Context(schwarz_tau=1e6).load(_shells(nd, n_p)).schwarz()
    assert (small > 0).all()
    assert (Q[:nd, :nd] == small[0, 1]).all()
    assert (Q[:nd, nd:] == small[0, 2]).all() and (Q[nd:, :nd] == small[0, 2]).all()
    assert (Q[nd:, nd:] == small[2, 3]).all()
