"""FP64 builds on strip tiles at the edges of their range: every fragment count
of a q-tile (n_omega up to 128, and two or more equal tiles beyond), odd and
even n_bf and n_omega (an odd row's last pair is staged one element early),
n_omega = n_mo = n_bf, one auxiliary function, k remainders, operands that do
not start 16-byte aligned, the smallest sizes (a one-orbital space takes the
register-staged tile), both tile widths, and the Fock step with its workspace
capped.

Tolerance: every output is a chain of FP64 contractions of at most
max(n_bf, n_aux, 2 n_omega) terms, each rounding at most 2^-53 of its sum of
magnitudes; normwise 1e-11 covers 4 of them at these sizes with a factor of
about 100 for cancellation, while a lost or repeated column costs 1e-3 or more.
"""
import numpy as np
import pytest

import synth
from gpu_util import host, relerr, to_dev
from oracle import pnof7_ri as ri

pytestmark = pytest.mark.gpu
TOL = 1e-11
KEYS = ("b_half", "b_mo", "d", "J", "K", "Jn", "Kn", "lam", "grad")


def check(ctx, inst, t=None):
    t = t or to_dev(inst)
    o = ctx.build(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], inst.n_pairs, inst.n_cwo)
    ctx.sync()
    ref = ri.build_instance(inst)
    for k in KEYS:
        assert relerr(host(o[k]), ref[k]) < TOL, k
    assert np.array_equal(host(o["Jn"]), host(o["Jn"]).transpose(0, 2, 1))
    return o, ref


@pytest.fixture(scope="module")
def ctx():
    import paper_2012_15662_amd as rif
    c = rif.Context()
    yield c
    c.close()


# n_omega: 1 (register tile), 2, then one size in and one past each 16-row fragment, and 129, 200, 257
@pytest.mark.parametrize("nb,na,npair,ncwo", [
    (2, 3, 1, 1), (3, 1, 1, 1), (3, 5, 1, 2), (16, 17, 4, 3), (17, 16, 17, 0), (33, 47, 11, 2), (48, 31, 16, 2), (49, 33, 7, 6), (65, 20, 13, 4),
    (81, 18, 27, 2), (97, 40, 16, 5), (113, 15, 28, 3), (128, 16, 32, 3), (131, 33, 43, 2), (201, 21, 40, 4), (260, 19, 257, 0),
])
@pytest.mark.parametrize("variant", [0, 1])
def test_sizes(ctx, nb, na, npair, ncwo, variant):
    if ncwo == 0:   # no weak orbitals: the pairing scheme needs one; use as many pairs as fit
        npair, ncwo = npair // 2, 1
    ctx.set_tile_variant(variant)
    try:
        check(ctx, synth.make_instance(nb, na, npair, ncwo, nb + na))
    finally:
        ctx.set_tile_variant(-1)


def test_transform_of_one_orbital(ctx):
    import torch
    rng = np.random.default_rng(1)
    for nb, na in ((1, 1), (1, 4), (5, 3), (37, 19)):
        b = rng.standard_normal((na, nb, nb))
        b = np.ascontiguousarray(b + b.transpose(0, 2, 1))
        C = np.linalg.qr(rng.standard_normal((nb, nb)))[0]
        bh, bmo, d = ctx.transform(torch.from_numpy(b).cuda(), torch.from_numpy(np.ascontiguousarray(C)).cuda(), 1)
        Jn, Kn = ctx.jk_ao_per_mo(torch.from_numpy(b).cuda(), bh, d)
        ctx.sync()
        r = ri.half_transform(b, C[:, :1])
        rd = ri.diag_of(ri.mo_transform(r, C[:, :1]))
        rJ, rK = ri.jk_ao_per_mo(b, r, rd)
        assert relerr(host(bh), r) < TOL and relerr(host(d), rd) < TOL
        assert relerr(host(Jn), rJ) < TOL and relerr(host(Kn), rK) < TOL


def test_unaligned_operands(ctx):
    """b, C and the outputs start 8 bytes past a 16-byte boundary."""
    import torch
    inst = synth.make_instance(67, 45, 9, 3, 5)
    t = to_dev(inst)

    def shifted(x):
        buf = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")
        buf[1:] = x.reshape(-1)
        return buf[1:].view(x.shape)
    u = {k: shifted(v) if v.dtype == torch.float64 else v for k, v in t.items()}
    out = ctx.outputs(67, 45, 9, 3, 67)
    out = {k: shifted(v) for k, v in out.items()}
    o = ctx.build(u["b"], u["C"], u["H"], u["occ"], u["pair_of"], 9, 3, out=out)
    ctx.sync()
    ref = ri.build_instance(inst)
    for k in KEYS:
        assert relerr(host(o[k]), ref[k]) < TOL, k


def test_fock_with_capped_workspace():
    """The Fock step's partials need more than its split sums at large n_bf:
    under a cap between the two it takes the register-staged tile."""
    import paper_2012_15662_amd as rif
    inst = synth.make_instance(400, 8, 100, 3, 6)
    t = to_dev(inst)
    ref = ri.build_instance(inst)
    c = rif.Context()
    o = c.build(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], 100, 3)
    c.sync()
    assert relerr(host(o["grad"]), ref["grad"]) < TOL
    c2 = rif.Context()
    c2.set_workspace_limit(60_000_000)   # 56 MB with split sums, 65 MB with the strips' partials
    o2 = c2.build(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], 100, 3)
    c2.sync()
    assert relerr(host(o2["grad"]), ref["grad"]) < TOL
    c.close()
    c2.close()
