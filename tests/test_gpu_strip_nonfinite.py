"""An infinity in b through the FP64 strip tiles: exactly the elements of b_half, b_mo,
d and J^q that a plain product makes infinite are infinite, and none is NaN, also
where an odd n_bf has its last pair staged one element early."""
import numpy as np
import pytest

from tests.gpu_util import host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [201, 200, 175, 193])
@pytest.mark.parametrize("back", [1, 2, 3])   # from the end of the row
def test_infinity_stays_one(nb, back):
    import torch
    import paper_2012_15662_amd as rif
    na, w, l0, x = 600, 48, 7, nb - back
    assert 3 * (-(-na // 8)) >= 192   # MO tiles on strips (three 16-orbital blocks)
    rng = np.random.default_rng(nb + back)
    b = rng.standard_normal((na, nb, nb))
    b = b + b.transpose(0, 2, 1)
    b[l0, x, x] = np.inf
    C = np.ascontiguousarray(np.linalg.qr(rng.standard_normal((nb, nb)))[0])
    ctx = rif.Context()
    tb = torch.from_numpy(b).cuda()
    bh, bmo, d = ctx.transform(tb, torch.from_numpy(C).cuda(), w)
    Jn, Kn = ctx.jk_ao_per_mo(tb, bh, d)
    ctx.sync()
    with np.errstate(invalid="ignore"):
        rh = np.where(np.arange(nb) == x, np.sign(C[x, :w])[:, None] * np.inf, 0.0)   # [q][nu] of l0
        rm = np.outer(C[x, :w], C[x, :w]) * np.inf
    for got, ref in ((host(bh)[:, l0], rh), (host(bmo)[l0], rm), (host(d)[l0], np.diag(rm))):
        assert not np.isnan(got).any()
        assert np.array_equal(np.isinf(got), np.isinf(ref))
        assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    for got, skip in ((host(bh), 1), (host(bmo), 0), (host(d), 0)):
        assert np.isfinite(np.delete(got, l0, axis=skip)).all()
    # J^q = sum_l d_lq b_l: every element takes d of l0, infinite with the sign of b's
    J = host(Jn)
    assert not np.isnan(J).any() and np.isinf(J).all()
    assert np.array_equal(np.sign(J[0]), np.sign(b[l0]))
    ctx.close()
