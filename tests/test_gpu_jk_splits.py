"""J and K (MO) at the sizes where the split over l and the reduction's tiles
change: one auxiliary function, a single element, few splits (a thread per
element), one and several chunks of 64 splits and their remainders; the
allocation-free call takes the same path.

Tolerance: sums of n_aux FP64 products, each step rounding at most 2^-53 of the
sum of magnitudes: n_aux 2^-53, against the largest element, which for K (a sum
of squares) and J's diagonal is at least the magnitude sum of its neighbours up
to the factor 4 allowed here.
"""
import numpy as np
import pytest

from gpu_util import host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nw", [(1, 1), (15, 2), (16, 3), (64, 4), (65, 4), (7, 1), (9, 2), (61, 5), (192, 10), (255, 16), (600, 48), (603, 47), (500, 99), (90, 130), (40, 300), (17, 520)])
def test_jk_mo_matches_numpy(na, nw):
    import torch
    import paper_2012_15662_amd as rif
    ctx = rif.Context(0)
    rng = np.random.default_rng(na * 1000 + nw)
    bmo = rng.standard_normal((na, nw, nw))
    bmo = (bmo + bmo.transpose(0, 2, 1)) / 2
    d = np.ascontiguousarray(np.diagonal(bmo, axis1=1, axis2=2))
    tb, td = torch.from_numpy(bmo).cuda(), torch.from_numpy(d).cuda()
    J, K = ctx.jk_mo(tb, td)
    J2, K2 = ctx.jk_mo_noalloc(tb, td, torch.full_like(J, np.nan), torch.full_like(K, np.nan))
    ctx.sync()
    tol = 4 * (na + 4) * 2.0 ** -53
    assert relerr(host(K), np.einsum("lpq,lpq->pq", bmo, bmo)) < tol
    assert relerr(host(J), d.T @ d) < tol
    assert np.array_equal(host(J), host(J2)) and np.array_equal(host(K), host(K2))
    ctx.close()
