"""The warm-start network's fused passes at the row counts where their split
changes: part of a 16-row workgroup, the 16/32-row switch, one and several
splits of the weight gradients, and an arena too small for the splits.

Tolerance: FP32 operands and activations with sums of at most 129 terms, each
rounding at most 2^-24 of the term sum: 129 * 2^-24 per layer, four layers
forward and three more (with the sum over rows in FP64 of 128-row FP32 parts)
backward; normwise over the array.
"""
import numpy as np
import pytest

from gpu_util import host, relerr
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu
LAYER = 129 * 2.0 ** -24
SWITCH = 256 * 48   # rows from which a workgroup takes 32


@pytest.mark.parametrize("rows,limit", [(1, 0), (15, 0), (16, 0), (17, 0), (127, 0), (129, 0), (260, 0), (SWITCH, 0), (SWITCH + 1, 0),
                                        (13001, 0), (6001, 300000), (13001, 500000)])
def test_passes_match_oracle(rows, limit):
    import torch
    import paper_2012_15662_amd as rif
    ctx = rif.Context(0)
    if limit:   # lp and dZ fit, the split partials and the third dA do not
        ctx.set_workspace_limit(limit)
    rng = np.random.default_rng(rows)
    th = (omlp.init_params(2) + 0.05 * rng.standard_normal(omlp.N_PARAMS)).astype(np.float32)
    X = rng.standard_normal((rows, omlp.N_IN)).astype(np.float32)
    M = np.ones((rows, omlp.N_OUT), np.float32)
    M[rng.random((rows, omlp.N_OUT)) < 0.3] = 0
    M[:, 0] = 1
    T = (rng.random((rows, omlp.N_OUT)) * M).astype(np.float32)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    f = dict(dtype=torch.float32, device="cuda")
    H, Z, P = torch.empty((3, rows, 128), **f), torch.empty((rows, 7), **f), torch.empty((rows, 7), **f)
    dA, g, loss = torch.empty((2, rows, 128), **f), torch.full((omlp.N_PARAMS,), np.nan, **f), torch.zeros(1, dtype=torch.float64, device="cuda")
    tX, tM, tT, tth = dev(X), dev(M), dev(T), dev(th)
    ctx.mlp_forward(tX, tM, tth, H, Z, P)
    ctx.mlp_backward(tX, tM, tT, tth, H, Z, dA, g, loss)
    ctx.sync()
    p, cache = omlp.forward(th.astype(np.float64), X.astype(np.float64), M.astype(np.float64))
    gr = omlp.backward(th.astype(np.float64), cache, T.astype(np.float64), M.astype(np.float64))
    assert relerr(host(H), np.stack(cache[1:4])) < 3 * LAYER
    assert relerr(host(P), p) < 4 * LAYER
    assert relerr(host(g), gr) < 7 * LAYER
    assert abs(host(loss)[0] - omlp.loss(p, T, M)) < 4 * LAYER * omlp.loss(p, T, M)
    ctx.close()


def test_tanh_saturates_and_keeps_nan():
    """Pre-activations from 1e-30 to infinity, and NaN, through one layer."""
    import torch
    import paper_2012_15662_amd as rif
    ctx = rif.Context(0)
    v = np.concatenate([np.geomspace(1e-30, 60.0, 60), -np.geomspace(1e-12, 30.0, 30), [0.0, 1e30, -1e30]]).astype(np.float32)
    rows = v.size + 1
    X = np.zeros((rows, omlp.N_IN), np.float32)
    X[:-1, 0] = v
    X[-1, 0] = np.nan
    th = np.zeros(omlp.N_PARAMS, np.float32)
    th[:128] = 1.0   # row 0 of W1
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    f = dict(dtype=torch.float32, device="cuda")
    H, Z, P = torch.empty((3, rows, 128), **f), torch.empty((rows, 7), **f), torch.empty((rows, 7), **f)
    ctx.mlp_forward(dev(X), dev(np.ones((rows, 7), np.float32)), dev(th), H, Z, P)
    ctx.sync()
    h = host(H)[0]
    ref = np.tanh(v.astype(np.float64))[:, None]
    assert np.all(np.abs(h[:-1] - ref) <= 2.0 ** -24 * (1 + 1e-4) * np.abs(ref))
    assert np.all(np.isnan(h[-1]))
    ctx.close()
