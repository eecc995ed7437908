"""The one-launch factorisation of rif_prepare_b at the edges of its layout:
panels (8, 12 and 16 positions), rows of one to four elements a thread (512 a
thread apart), and the sizes past which the per-column launches take over.

Each is checked by its backward error: elementwise, |G[perm][:, perm] - L D L^T|
is at most c n u |L| |D| |L^T| for any pivot sequence (Higham, Accuracy and
Stability of Numerical Algorithms, theorem 11.3, whose constant is a low-degree
polynomial of n; 4 n u is taken, with twice as much for the product here).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2012_15662_amd as rif
    c = rif.Context()
    yield c
    c.close()


def metric(kind, n):
    rng = np.random.default_rng(n)
    if kind == "ties":      # small integers: many equal candidates, exact zeros
        G = rng.integers(-2, 3, (n, n)).astype(float)
        return G + G.T
    X = rng.standard_normal((n, n))
    if kind == "indefinite":    # interchanges and 2x2 blocks throughout
        return X + X.T
    d = 10.0 ** rng.uniform(-2, 2, n)   # badly scaled: the second pivot test at most columns
    G = (X @ X.T / n + 0.1 * np.eye(n)) * d * d[:, None]
    return (G + G.T) / 2


SIZES = [1, 2, 15, 16, 17, 33, 255, 257, 511, 512, 513, 1024, 1025, 1537, 2048, 2049]


@pytest.mark.parametrize("n,kind", [(n, k) for n in SIZES for k in ("scaled", "indefinite", "ties")
                                    if k != "ties" or n < 600])
def test_factorisation_backward_error(ctx, n, kind):
    import torch
    print("case factorise:", n, kind, flush=True)
    G = metric(kind, n)
    T = torch.ones((n, 1, 1), dtype=torch.float64, device="cuda")
    _, perm, L, D, _ = ctx.prepare_b(T, torch.from_numpy(G).cuda(), factors=True)
    ctx.sync()
    perm, L, D = perm.cpu().numpy(), L.cpu().numpy(), D.cpu().numpy()
    assert np.array_equal(np.sort(perm), np.arange(n))
    assert np.array_equal(np.triu(L), np.eye(n))
    off = np.abs(np.diagonal(D, 1)) > 0
    assert not np.any(off[1:] & off[:-1])          # blocks of one or two
    assert np.array_equal(D, np.tril(np.triu(D, -1), 1)) and np.array_equal(D, D.T)
    assert not np.any(np.diagonal(L, -1)[off])     # L is I on a 2x2 block
    err = np.abs(G[np.ix_(perm, perm)] - L @ D @ L.T)
    bound = 8 * n * U * (np.abs(L) @ np.abs(D) @ np.abs(L).T)
    assert np.all(err <= bound), (err / np.maximum(bound, 1e-300)).max()


@pytest.mark.parametrize("n,n_bf", [(1, 1), (1, 5), (2, 2), (3, 1), (3, 3), (15, 16), (16, 17), (17, 15), (31, 8),
                                    (64, 9), (65, 33), (127, 24), (129, 31), (144, 48), (257, 50), (300, 113)])
def test_solve_matches_float64(ctx, n, n_bf):
    """The solve at the edges of its tiles (rows of 16 to 128, blocks of 8 x 16
    pairs, odd sizes).  With X = L^-1, computed by substitution, the inverse is
    wrong by at most c n u |X| |L| |X| and the sum over i by n u |M'| |T|, which is
    no larger: 8 n u of the first bounds both and the reference's own rounding."""
    import torch
    print("case solve:", n, n_bf, flush=True)
    rng = np.random.default_rng(7 * n + n_bf)
    G = rng.standard_normal((n, n)) * (0.3 / n ** 0.5)
    G = np.diag(rng.uniform(0.5, 2.0, n)) + (G + G.T) * 0.2
    T = rng.standard_normal((n, n_bf, n_bf))
    T = T + T.transpose(0, 2, 1)
    b, perm, L, D, nr = ctx.prepare_b(torch.from_numpy(T).cuda(), torch.from_numpy(G).cuda(), factors=True)
    ctx.sync()
    b, perm, L, D = b.cpu().numpy(), perm.cpu().numpy(), L.cpu().numpy(), D.cpu().numpy()
    d = np.diagonal(D)
    assert int(nr.cpu()[0]) == 0 and np.array_equal(D, np.diag(d)) and np.all(d > 0)
    X = np.linalg.inv(L)
    Tp = T[perm].reshape(n, -1)
    ref = ((X / np.sqrt(d)[:, None]) @ Tp).reshape(b.shape)
    bound = 8 * n * U * (np.abs(X) @ np.abs(L) @ np.abs(X) / np.sqrt(d)[:, None]) @ np.abs(Tp)
    assert np.all(np.abs(b - ref).reshape(n, -1) <= np.maximum(bound, 8 * U * np.abs(Tp).max()))
    assert np.array_equal(b, b.transpose(0, 2, 1))
