"""The occupation-number optimiser's iterates against the same L-BFGS (history 8,
backtracking from a unit step with the Armijo test) in numpy on the oracle's energy
and gradient: variables after a few iterations and after the history's ring has
wrapped, in both kernels (up to 128 orbitals in Omega and above).

Tolerance: a run whose start is off by 1e-15 differs from an undisturbed one by at
most AMPLIFY x 1e-15 in the numpy optimiser at the iteration compared, over these problems;
the kernels' roundings (fused, other sums) act like some hundred such disturbances.
A wrong scalar product or history entry moves the variables by 1e-3 and more.
"""
import numpy as np
import pytest

from oracle import on_opt as oon
from tests.gpu_util import host
from tests.test_gpu_on_sizes import problem

SIZES = [(2, 3), (13, 4), (8, 14), (64, 1), (32, 3), (43, 2), (65, 1), (10, 14)]   # pairs, weak a pair
AMPLIFY = {1: 1e1, 3: 1e2, 12: 1e4}


def evaluate(x, H, J, K, pair, npair, m):
    n = oon.gamma_to_n(x, pair, npair, m)
    return oon.energy_n(n, H, J, K, pair, npair), oon.dn_dgamma(x, pair, npair, m).T @ gradient(n, H, J, K, pair, npair)


def gradient(n, H, J, K, pair, npair):
    """oracle.on_opt.grad_n by rows."""
    phi = np.sqrt(n * (1 - n))
    dphi = (1 - 2 * n) / (2 * np.maximum(phi, 1e-300))
    same = pair[:, None] == pair[None, :]
    weak = np.arange(len(n)) >= npair
    sg = np.where(weak[:, None] & weak[None, :], 1.0, -1.0)
    own = sg * np.sqrt(n[None, :] / np.maximum(n[:, None], 1e-300)) * K
    np.fill_diagonal(own, 0.0)
    other = 2 * (2 * n[None, :] * J + (-n[None, :] - np.outer(dphi, phi)) * K)
    return 2 * H + np.diag(K) + np.where(same, own, other).sum(1)


def iterate(x, steps, args):
    E, g = evaluate(x, *args)
    S, Y = [], []
    for _ in range(steps):
        gm = np.max(np.abs(g))
        d, al = g.copy(), []
        for s, y in reversed(list(zip(S, Y))):
            al.append(s @ d / (s @ y))
            d -= al[-1] * y
        d *= (S[-1] @ Y[-1]) / (Y[-1] @ Y[-1]) if S else min(1.0, 1.0 / gm)
        for s, y, a in zip(S, Y, reversed(al)):
            d += (a - y @ d / (s @ y)) * s
        d = -d
        if not g @ d < 0:
            d, S, Y = -g * min(1.0, 1.0 / gm), [], []
        step = 1.0
        while True:
            En, gn = evaluate(x + step * d, *args)
            if En <= E + 1e-4 * step * (g @ d):
                break
            step *= 0.5
            assert step > 1e-6
        xn = x + step * d
        if (xn - x) @ (gn - g) > 1e-300:
            S, Y = (S + [xn - x])[-8:], (Y + [gn - g])[-8:]
        x, E, g = xn, En, gn
    return x


def cases():
    for s in SIZES:
        for shuffled in (False, True):
            yield s, problem(*s, shuffled)


def test_numpy_gradient_is_the_oracles():
    for (npair, m), (H, J, K, pair) in list(cases())[:4]:
        n = oon.gamma_to_n(oon.cold_start(npair, m), pair, npair, m)
        ref = oon.grad_n(n, H, J, K, pair, npair)
        assert np.max(np.abs(gradient(n, H, J, K, pair, npair) - ref)) < 1e-12 * np.max(np.abs(ref))


@pytest.mark.parametrize("steps", sorted(AMPLIFY))
def test_disturbed_start(steps):
    """AMPLIFY holds in the numpy optimiser."""
    rng = np.random.default_rng(3)
    worst = 0.0
    for (npair, m), (H, J, K, pair) in cases():
        args = (H, J, K, pair, npair, m)
        x0 = oon.cold_start(npair, m)
        x = iterate(x0, steps, args)
        y = iterate(x0 + 1e-15 * rng.choice([-1.0, 1.0], len(x0)), steps, args)
        worst = max(worst, np.max(np.abs(x - y)) / 1e-15)
    print(steps, worst)
    assert worst < AMPLIFY[steps]


@pytest.mark.gpu
@pytest.mark.parametrize("steps", sorted(AMPLIFY))
def test_iterates(steps):
    import torch
    import paper_2012_15662_amd as rif
    ctx = rif.Context()
    data = list(cases())
    probs = [tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in d) + s for s, d in data]
    onset = rif.OnSet(ctx, probs, tol=1e-13, max_it=steps)
    x0 = [oon.cold_start(*s) for s, _ in data]
    for k, x in enumerate(x0):
        onset.gamma[onset.gslices[k]] = torch.from_numpy(x).cuda()
    ctx.on_optimize(onset)
    ctx.sync()
    gam, it = host(onset.gamma), host(onset.iters)
    for k, ((npair, m), (H, J, K, pair)) in enumerate(data):
        ref = iterate(x0[k], steps, (H, J, K, pair, npair, m))
        err = np.max(np.abs(gam[onset.gslices[k]] - ref))
        print("case on path:", npair, m, "steps", steps, "error", err, flush=True)
        assert it[k] == steps
        assert err < 100 * AMPLIFY[steps] * 1e-15, (npair, m)
    ctx.close()
