"""The preparation with no room for the one-launch factorisation's slots: column by
column, with the same pivots and the same b.

Tolerance: both run the same steps on a metric of condition about 1e2 (diagonal
blocks, with interchanges and 2x2 blocks); their roundings differ by n_aux 2^-53
times the condition, 6e-12 at n_aux 520."""
import numpy as np
import pytest

from tests.gpu_util import host, relerr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nb", [(1, 1), (2, 3), (65, 9), (520, 14)])
def test_limited_arena(n, nb):
    import torch
    import paper_2012_15662_amd as rif
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    w = np.geomspace(1.0, 1e-2, n) * np.where(np.arange(n) % 3 == 1, -1.0, 1.0)
    G = torch.from_numpy(np.ascontiguousarray((Q * w) @ Q.T)).cuda()
    G = (G + G.T) / 2
    T = torch.from_numpy(rng.standard_normal((n, nb, nb))).cuda()
    T = T + T.transpose(1, 2)
    c, small = rif.Context(), rif.Context()
    # every matrix begins at a multiple of 256 bytes
    small.set_workspace_limit(6 * ((8 * n * n + 255) // 256 * 256) + 16 * n + 6 * 256)
    one = c.prepare_b(T.contiguous(), G.contiguous(), factors=True)
    two = small.prepare_b(T.contiguous(), G.contiguous(), factors=True)
    c.sync()
    small.sync()
    assert np.array_equal(host(one[1]), host(two[1])) and host(one[4])[0] == host(two[4])[0]
    for k in (0, 2, 3):
        assert relerr(host(two[k]), host(one[k])) < 6e-12, k
    c.close()
    small.close()
