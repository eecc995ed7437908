"""The occupation-number optimiser at the edges of its two kernels: one problem in
the registers of a workgroup up to 128 orbitals in Omega, the general kernel above,
and pair maps in any order.

The energy returned is the oracle's at the returned variables, to the 1e-12 of the
sum's rounding (n^2 terms of O(1) magnitude, n <= 160, against |E| of their order),
and the point is stationary to the optimiser's own tolerance.
"""
import numpy as np
import pytest

from oracle import on_opt as oon
from tests.gpu_util import host

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 14), (2, 3), (8, 7), (13, 4), (8, 14), (64, 1), (32, 3), (65, 1), (10, 14)]   # pairs, weak a pair


def problem(npair, m, shuffled):
    rng = np.random.default_rng(100 * npair + m)
    w = npair * (1 + m)
    b = rng.standard_normal((3 * w, w, w)) * (0.5 / w) ** 0.5
    b = b + b.transpose(0, 2, 1)
    d = np.einsum("kpp->kp", b)
    J, K = d.T @ d, (b * b).sum(0)
    H = np.sort(rng.standard_normal(w)) - 2.0
    pair = np.concatenate([np.arange(npair), np.repeat(np.arange(npair), m)])
    if shuffled:
        pair[npair:] = rng.permutation(pair[npair:])
    return H, J, K, pair.astype(np.int32)


@pytest.mark.parametrize("shuffled", [False, True])
def test_energy_and_stationarity(shuffled):
    import torch
    import paper_2012_15662_amd as rif
    from paper_2012_15662_amd import warmstart as ws
    ctx = rif.Context()
    data = [problem(p, m, shuffled) for p, m in SIZES]
    probs = [tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in d) + s for d, s in zip(data, SIZES)]
    onset = rif.OnSet(ctx, probs, tol=1e-8, max_it=400)
    it, st, _ = ws.solve(ctx, onset, ws.prior_rows(onset))
    E, gam, occ = host(onset.energy), host(onset.gamma), host(onset.occ)
    for k, ((H, J, K, pair), (npair, m)) in enumerate(zip(data, SIZES)):
        print("case on sizes:", npair, m, "iterations", it[k], "status", st[k], flush=True)
        x = gam[onset.gslices[k]]
        ref = oon.energy_gamma(x, H, J, K, pair, npair, m)
        assert abs(E[k] - ref) <= 1e-12 * abs(ref)
        n = oon.gamma_to_n(x, pair, npair, m)
        assert np.max(np.abs(occ[onset.oslices[k]] - n)) <= 1e-14
        assert st[k] in (0, 1, 2)
        if st[k] == 0:
            assert np.max(np.abs(oon.grad_gamma(x, H, J, K, pair, npair, m))) < 1e-7
    assert np.mean(st == 0) >= 0.5
    ctx.close()


def test_strong_orbital_outside_its_pair():
    """Two strong orbitals whose map entries are exchanged: energy and ONs as the
    oracle has them for that map."""
    import torch
    import paper_2012_15662_amd as rif
    from paper_2012_15662_amd import warmstart as ws
    ctx = rif.Context()
    H, J, K, pair = problem(6, 3, False)
    pair[[0, 4]] = pair[[4, 0]]
    onset = rif.OnSet(ctx, [tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (H, J, K, pair)) + (6, 3)])
    ws.solve(ctx, onset, ws.prior_rows(onset))
    x = host(onset.gamma)
    ref = oon.energy_gamma(x, H, J, K, pair, 6, 3)
    assert abs(host(onset.energy)[0] - ref) <= 1e-12 * abs(ref)
    ctx.close()
