"""A build captured with autotuning on and tile choices saved when the FP64 steps had
four variants each: nothing is timed into the graph, and every replay (with eager
work between) equals the eager build of the default choices bit for bit."""
import numpy as np
import pytest

import synth
from tests.gpu_util import host, to_dev

pytestmark = pytest.mark.gpu
KEYS = ("b_half", "b_mo", "d", "J", "K", "Jn", "Kn", "energy", "lam", "grad")


@pytest.mark.parametrize("saved", [True, False])
def test_capture_with_saved_choices(saved):
    import torch
    import paper_2012_15662_amd as rif
    inst = synth.make_instance(130, 259, 7, 3, 21)
    t = to_dev(inst)
    w = inst.n_omega
    s = torch.cuda.Stream()
    ctx = rif.Context(stream=s)
    try:
        with torch.cuda.stream(s):
            out = ctx.build(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], inst.n_pairs, inst.n_cwo)
        torch.cuda.synchronize()
        eager = {k: host(out[k]).copy() for k in KEYS}
        if saved:
            ms = " | 0.1 0.1 0.1 0.1\n"
            ctx.tune_load(f"half_transform 0 130 {130 * 259} {w} 130 -> 2{ms}mo_transform 0 130 259 {w} 130 -> 3{ms}"
                          f"jao 0 130 259 {w} -> 3{ms}fock 0 130 {w} 130 64 -> 0{ms}")
        ctx.autotune(True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ctx.build(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], inst.n_pairs, inst.n_cwo, out=out)
        torch.cuda.synchronize()
        for rep in range(3):
            for k in KEYS:
                out[k].fill_(float("nan"))
            x = torch.randn(512, 512, device="cuda")
            y = (x @ x).sum()
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            for k in KEYS:
                assert np.array_equal(host(out[k]), eager[k]), (rep, k)
            del y
        del g
    finally:
        ctx.close()
