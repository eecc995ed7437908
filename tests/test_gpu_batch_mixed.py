"""FP64 batches of molecules that rif_build gives different kernels: some below and
some above the size from which the MO transform runs on strips, and one whose slabs
strips do not take at all.  Each molecule's results equal its single build's bit for
bit (with a tile variant set and with the library's own choice, launched and as a
graph), and the oracle's to 1e-11 normwise (chains of FP64 contractions of at most
max(n_bf, n_aux, 2 n_omega) terms, each rounding at most 2^-53 of its sum of
magnitudes; a lost column costs 1e-3 or more).
"""
import numpy as np
import pytest

import synth
from oracle import pnof7_ri as ri
from tests.gpu_util import host, relerr, to_dev

pytestmark = pytest.mark.gpu
KEYS = ("b_half", "b_mo", "d", "J", "K", "Jn", "Kn", "energy", "lam", "grad")
SMALL = [(61, 183, 5, 2, 71), (100, 300, 8, 2, 72), (37, 111, 3, 2, 73)]
LARGE = [(160, 520, 43, 2, 74), (201, 603, 16, 2, 75), (143, 515, 14, 4, 76), (175, 703, 23, 4, 77)]


def mo_tiles(nb, na, npair, ncwo, seed=0):
    w = npair * (1 + ncwo)
    return sum(-(-16 * (p + 1) // 128) for p in range(-(-w // 16))) * -(-na // 8)


@pytest.fixture(scope="module")
def ctx():
    import paper_2012_15662_amd as rif
    c = rif.Context()
    yield c
    c.close()


@pytest.fixture(scope="module")
def molecules():
    got = {}
    for s in SMALL + LARGE:
        inst = synth.make_instance(*s)
        got[s] = (inst, to_dev(inst), ri.build_instance(inst))
    return got


@pytest.mark.parametrize("variant", [-1, 0, 1])
@pytest.mark.parametrize("shapes", [SMALL + LARGE, LARGE, [LARGE[1], SMALL[0]]], ids=["both", "strips", "one_each"])
def test_batch_equals_single(ctx, molecules, shapes, variant):
    assert all(mo_tiles(*s) < 192 for s in SMALL) and all(mo_tiles(*s) >= 192 for s in LARGE)
    ctx.set_tile_variant(variant)
    try:
        items = [(molecules[s][1], s[2], s[3], None) for s in shapes]
        batch = ctx.batch(items)
        singles = [{k: host(v).copy() for k, v in ctx.build_instance(t, npair, ncwo).items()} for t, npair, ncwo, _ in items]
        for graph in (False, True, True):
            for out in batch.outs:
                for k in KEYS:
                    out[k].fill_(float("nan"))
            batch.run(use_graph=graph)
            ctx.sync()
            for s, single, out in zip(shapes, singles, batch.outs):
                for k in KEYS:
                    assert np.array_equal(host(out[k]), single[k]), (s, k, graph)
                for k in KEYS:
                    ref = np.atleast_1d(molecules[s][2][k])
                    assert relerr(single[k], ref) < 1e-11, (s, k)
        batch.close()
    finally:
        ctx.set_tile_variant(-1)


def test_batch_with_a_molecule_past_the_strips(ctx, molecules):
    import torch
    nb, na, w = 5900, 3, 4
    print(f"case batch with n_bf {nb}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    r = lambda *s: torch.randn(s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    b = r(na, nb, nb) * nb ** -0.5
    b = (b + b.transpose(1, 2)).contiguous()
    H = r(nb, nb)
    big = {"b": b, "C": torch.linalg.qr(r(nb, w))[0].contiguous(), "H": H + H.T,
           "occ": torch.tensor([0.9375, 0.875, 0.125, 0.0625], dtype=torch.float64, device="cuda"),
           "pair_of": torch.tensor([0, 1, 1, 0], dtype=torch.int32, device="cuda")}
    s = LARGE[1]
    items = [(molecules[s][1], s[2], s[3], None), (big, 2, 1, None)]
    batch = ctx.batch(items)
    batch.run(use_graph=False)
    ctx.sync()
    for (t, npair, ncwo, _), out in zip(items, batch.outs):
        single = ctx.build_instance(t, npair, ncwo)
        ctx.sync()
        for k in KEYS:
            assert torch.equal(out[k], single[k]), (npair, k)
    batch.close()
