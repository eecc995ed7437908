"""FP64 steps at the largest slabs that strip tiles take, where 16 rows of one n_bf^2
slab each reach the end of 32-bit offsets: a build at odd n_bf 5795 with 17
auxiliary functions and 16 orbitals (two k slices in J^q, one in each half of the
Fock step), against plain torch products in FP64; and the preparation's solve where
one slab passes 2^32 bytes.

Tolerance: chains of FP64 contractions of at most n_bf terms, each rounding at most
2^-53 of its sum of magnitudes: normwise 1e-11 covers them with a factor of 10 and
more; a column read from the wrong row costs 1e-2.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 1e-11


def err(got, ref):
    return float((got - ref).abs().max() / ref.abs().max())


def symmetric(nb, scale, gen):
    import torch
    x = torch.randn((nb, nb), dtype=torch.float64, device="cuda", generator=gen)
    return (x + x.T) * (0.5 * scale)


def test_build_at_the_largest_slabs():
    import torch
    import paper_2012_15662_amd as rif
    nb, na, npair, ncwo, w = 5795, 17, 8, 1, 16
    print(f"case n_bf {nb}, n_aux {na}, n_omega {w}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    b = torch.empty((na, nb, nb), dtype=torch.float64, device="cuda")
    for l in range(na):
        b[l] = symmetric(nb, nb ** -0.5, gen)
    H = symmetric(nb, 1.0, gen)
    C = torch.linalg.qr(torch.randn((nb, w), dtype=torch.float64, device="cuda", generator=gen))[0].contiguous()
    pm = np.concatenate([np.arange(npair), np.arange(npair)[::-1]]).astype(np.int32)
    occ = torch.cat([torch.full((npair,), 0.9375), torch.full((npair,), 0.0625)]).double().cuda()
    ctx = rif.Context()
    o = ctx.build(b, C, H, occ, torch.from_numpy(pm).cuda(), npair, ncwo)
    ctx.sync()
    bh = torch.stack([b[l] @ C for l in range(na)]).permute(2, 0, 1).contiguous()
    bmo = torch.stack([bh[:, l] @ C for l in range(na)])
    d = torch.diagonal(bmo, dim1=1, dim2=2).contiguous()
    for k, ref in (("b_half", bh), ("b_mo", bmo), ("d", d), ("J", d.T @ d), ("K", (bmo * bmo).sum(0))):
        assert err(o[k], ref) < TOL, k
    # PNOF7 coefficients: 2 n n J - (n n + phi phi) K between pairs, -sqrt(n n) K in one
    n = occ
    p = torch.from_numpy(pm).cuda().long()
    same = p[:, None] == p[None, :]
    phi, nn = torch.sqrt(n * (1 - n)), torch.outer(n, n)
    A = torch.where(same, torch.zeros_like(nn), 2 * nn)
    B = torch.where(same, -torch.sqrt(nn), -nn - torch.outer(phi, phi))
    B = torch.where(torch.eye(w, dtype=torch.bool, device="cuda"), n[:, None].expand(w, w), B)
    Y = (H @ C) * n
    for q in range(w):
        Jq = sum(d[l, q] * b[l] for l in range(na))
        assert err(o["Jn"][q], Jq) < TOL, ("Jn", q)
        Kq = bh[q].T @ bh[q]
        assert err(o["Kn"][q], Kq) < TOL, ("Kn", q)
        Y += Jq @ (C * A[:, q]) + Kq @ (C * B[:, q])
    assert err(o["lam"], C.T @ Y) < TOL
    ctx.close()


def test_prepare_with_slabs_past_32_bits():
    import torch
    import paper_2012_15662_amd as rif
    nb, n = 23201, 3
    print(f"case prepare n_bf {nb}, n_aux {n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    T = torch.empty((n, nb, nb), dtype=torch.float64, device="cuda")
    for k in range(n):
        T[k] = symmetric(nb, 1.0, gen)
    G = np.array([[4.0, 0.5, -0.25], [0.5, 3.0, 0.75], [-0.25, 0.75, 2.0]])   # no interchange: b^T = chol(G)^-1 T
    M = np.linalg.inv(np.linalg.cholesky(G))
    ctx = rif.Context()
    b = ctx.prepare_b(T, torch.from_numpy(G).cuda())
    ctx.sync()
    for k in range(n):
        for r in range(0, nb, 2048):
            ref = sum(float(M[k, i]) * T[i, r:r + 2048] for i in range(n))
            assert err(b[k, r:r + 2048], ref) < 1e-13, (k, r)
    ctx.close()
