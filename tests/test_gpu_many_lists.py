"""More than a thousand ket lists.

A context keeps one ket list per pair class, primitive count and set of rows
or windows.  Contractions of 1 to 16 primitives give 97 primitive-pair counts
in each of the six pair classes, and above 2048 functions a class is in up to
three sets.  The molecule is one centre with such shells beside single d
shells, each too far from everything for a pair; with a density on the centre
alone, the centre's block of J and K is that of the centre loaded alone (one
set of lists).  Very sharp s, p and d shells and a threshold between their
bounds and the others' leave few quartets, some of them in the last lists.
Tolerance as between summation orders elsewhere: 1e-12 of the largest element.
"""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


TAU = 20.0   # bounds of the sharp pairs: some 100, of the others: some 1


def _centre():
    shells = []
    for l in (0, 1, 2):
        for n in range(1, 17):
            ex = 0.6 * 1.15 ** np.arange(n)
            shells.append(W.Shell(0, l, ex, 1.0 / (1.0 + np.arange(n))))
        shells.append(W.Shell(0, l, 1e8 * 1.15 ** np.arange(16), 1.0 / (1.0 + np.arange(16))))
    return W.Molecule(np.array([2], dtype=np.int32), np.zeros((1, 3)), shells)


def _lists(m, Q):
    """Ket lists of a molecule above 2048 functions: s-s to d-s pairs are in three sets, d-p pairs in two."""
    sets = {(0, 0): 3, (1, 0): 3, (1, 1): 3, (2, 0): 3, (2, 1): 2, (2, 2): 1}
    seen = set()
    for a, u in enumerate(m.shells):
        for b, v in enumerate(m.shells[:a + 1]):
            if Q[a, b] * Q.max() >= TAU:
                seen.add((max(u.l, v.l), min(u.l, v.l), len(u.exps) * len(v.exps)))
    return sum(sets[x[:2]] for x in seen)


def _with_far_shells(m, n):
    xyz = np.concatenate([m.xyz, 200.0 + 100.0 * np.array([(i % 7, i // 7 % 7, i // 49) for i in range(n)])])
    far = [W.Shell(1 + i, 2, np.array([0.8]), np.array([1.0])) for i in range(n)]
    return W.Molecule(np.concatenate([m.Z, np.zeros(n, dtype=np.int32)]), xyz, m.shells + far)


@pytest.mark.parametrize("form", [0, 1])
def test_lists_of_every_contraction_and_set(form):
    import torch
    from paper_1708_00033_amd import hfx
    small = _centre()
    big = _with_far_shells(small, 320)
    n, N = small.nbf, big.nbf
    assert n == 170 and N > 2048
    s = torch.cuda.current_stream().cuda_stream
    D = torch.tensor(W.random_symmetric(n, 9, 0.1), device="cuda")
    DN = torch.zeros((N, N), dtype=torch.float64, device="cuda")
    DN[:n, :n] = D
    ca, cb = hfx.Context(schwarz_tau=TAU).load(small), hfx.Context(schwarz_tau=TAU).load(big)
    assert _lists(small, ca.schwarz()) > 1024
    cb.set_class_tuning(-1, 0, -1, form, -1)
    G, GN = torch.empty_like(D), torch.empty_like(DN)
    for cj, ck in ((1.0, 0.0), (0.0, -1.0)):
        ca.build_2e_dev(D.data_ptr(), cj, ck, G.data_ptr(), s)
        cb.build_2e_dev(DN.data_ptr(), cj, ck, GN.data_ptr(), s)
        torch.cuda.synchronize()
        assert (GN[:n, :n] - G).abs().max().item() <= 1e-12 * G.abs().max().item(), (cj, ck)
