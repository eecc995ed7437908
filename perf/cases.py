"""Performance cases of the RI-PNOF7 library: the work a program has it do, through its public entry points.

A case names an entry point ("what") and the sizes and options of one call.  Inputs follow the seeded recipe of the
repository's synthetic molecules: b[l] = (G + G^T)/2 exp(-3 l / n_aux) with G ~ N(0, 1/n_bf), orthonormal C, a
symmetric Gaussian H, strong occupations U(0.9, 0.99) with the rest of each pair shared by its weak orbitals.

  build    rif_build: every step of one build (an inner iteration that keeps J^q and K^q)
  direct   rif_build_direct: energy, Lagrangian and gradient only (an inner iteration of the orbital loop)
  batch    rif_batch_run: uneven molecules in one grouped graph replay
  prepare  rif_prepare_b: b from the three-centre integrals and the metric, once per molecule
  orbital  rif_orbital_step: one diagonalisation of F^lambda and the rotation of C
  on       rif_on_warmstart + rif_on_optimize: the occupation step of many molecules at once
  train    rif_mlp_forward + rif_mlp_backward + rif_adam: one epoch of the warm-start network
  loop     rif_pnof_optimize: one outer iteration with a few inner ones, start to end

"tune" stands for a program that lets the library time its tiles (rif_autotune) before its iterations start; the others
take the library's default choice.
"""
import math

import numpy as np
import torch

import paper_2012_15662_amd as rif

DEV = "cuda"
PREC = {"fp64": rif.FP64, "fp32": rif.FP32, "bf16x3": rif.BF16X3, "bf16x6": rif.BF16X6, "fp16x3": rif.FP16X3}
PIECES = {"bf16x3": 2, "bf16x6": 3, "fp16x3": 2}
OUT = ("b_half", "b_mo", "d", "J", "K", "Jn", "Kn", "energy", "lam", "grad")
N_IN, N_HID, N_OUT = 39, 128, 7


def _mol(n_bf, n_aux, n_pairs, n_cwo, **more):
    return dict({"n_bf": n_bf, "n_aux": n_aux, "n_pairs": n_pairs, "n_cwo": n_cwo}, **more)


def listed():
    return [
        # the oracle-sized molecule: launches and latency
        dict(_mol(48, 192, 5, 1, prec="fp64", presplit=False, tune=False), name="build_tiny", what="build"),
        # an odd basis size from the middle of the many-molecule range (n_aux = 3 n_bf, n_bf // 12 pairs, Ncwo 2)
        dict(_mol(201, 603, 16, 2, prec="fp64", presplit=False, tune=False), name="build_odd", what="build"),
        # cyclohexane-like: the headline workload, tuned as the benchmark runs it
        dict(_mol(348, 1044, 24, 4, prec="fp64", presplit=False, tune=True), name="build_c6h12", what="build"),
        # cyclodecane-like: n_omega = 200 is no multiple of the matrix tiles
        dict(_mol(580, 1740, 40, 4, prec="fp64", presplit=False, tune=True), name="build_c10h20", what="build"),
        # the reduced-precision mode that meets the 1 uEh target at every size, b stored once in its pieces
        dict(_mol(348, 1044, 24, 4, prec="bf16x6", presplit=True, tune=True), name="build_bf16x6", what="build"),
        # the orbital loop's build at the middle size of the scaling study
        dict(_mol(288, 864, 20, 4, prec="fp64", presplit=False, tune=False), name="direct_288", what="direct"),
        # many uneven molecules at once
        {"name": "batch_16", "what": "batch", "n_mol": 16, "lo": 60, "hi": 400, "sizes": 3, "n_cwo": 2, "prec": "fp64"},
        # the preparation the benchmark times: condition 1e10, three slightly negative eigenvalues
        {"name": "prepare_c6h12", "what": "prepare", "n_bf": 348, "n_aux": 1044, "cond": 1e10, "negative": 3},
        # one orbital step at the cyclohexane-like size
        {"name": "orbital_348", "what": "orbital", "n_bf": 348, "n_mo": 348, "n_omega": 120},
        # the held-out set of the warm-start study: 200 molecules, cold start
        {"name": "on_200", "what": "on", "n_mol": 200, "lo": 48, "hi": 200, "sizes": 11},
        # an epoch over the training set of the warm-start study
        {"name": "train_19553", "what": "train", "rows": 19553},
        # a whole call on the small molecule: one outer iteration, eight inner ones
        dict(_mol(48, 192, 5, 1, inner=8), name="loop_tiny", what="loop"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_mol(rng, top):
    """Sizes of the cycloalkane-like and many-molecule workloads: n_aux about 3 n_bf, n_bf // 12 to n_bf // 15 pairs, Ncwo 1..4."""
    n_bf = _log(rng, 48, top)
    n_pairs = max(2, n_bf // rng.randint(12, 15))
    return _mol(n_bf, int(n_bf * rng.uniform(2.6, 3.4)), n_pairs, rng.randint(1, 4))


def draw(rng):
    what = rng.choice(["build"] * 5 + ["direct"] * 2 + ["batch", "prepare", "orbital", "on", "train", "loop"])
    if what == "build":
        prec = rng.choice(["fp64"] * 4 + ["fp32", "bf16x6", "fp16x3", "bf16x3"])
        return dict(_draw_mol(rng, 480), what=what, prec=prec, presplit=prec != "fp64" and rng.random() < 0.5, tune=rng.random() < 0.5)
    if what == "direct":
        prec = rng.choice(["fp64"] * 3 + ["bf16x6"])
        return dict(_draw_mol(rng, 480), what=what, prec=prec, presplit=prec != "fp64", tune=rng.random() < 0.5)
    if what == "batch":
        lo = rng.randint(48, 120)
        return {"what": what, "n_mol": rng.randint(3, 16), "lo": lo, "hi": lo + rng.randint(20, 240), "sizes": rng.randrange(1 << 16),
                "n_cwo": rng.randint(1, 3), "prec": rng.choice(["fp64", "fp64", "bf16x6"])}
    if what == "prepare":
        n_bf = _log(rng, 40, 340)
        return {"what": what, "n_bf": n_bf, "n_aux": int(n_bf * rng.uniform(2.6, 3.1)), "cond": 10.0 ** rng.randint(4, 10), "negative": rng.choice([0, 3])}
    if what == "orbital":
        n = _log(rng, 20, 580)
        return {"what": what, "n_bf": n, "n_mo": n - rng.choice([0, 0, 1, 5]), "n_omega": max(2, n // 3)}
    if what == "on":
        lo = rng.randint(48, 90)
        return {"what": what, "n_mol": _log(rng, 1, 200), "lo": lo, "hi": lo + rng.randint(20, 110), "sizes": rng.randrange(1 << 16)}
    if what == "train":
        return {"what": what, "rows": _log(rng, 40, 19500)}
    n_bf = _log(rng, 24, 140)
    return dict(_mol(n_bf, 3 * n_bf + rng.randint(0, 40), max(2, n_bf // 12), rng.randint(1, 3), inner=rng.randint(3, 8)), what=what)


# ---- inputs ------------------------------------------------------------------
def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + salt)
    return g


def _pair_map(n_pairs, n_cwo):
    pm = np.empty(n_pairs * (1 + n_cwo), dtype=np.int32)
    pm[:n_pairs] = np.arange(n_pairs)
    for g in range(n_pairs):
        w = n_pairs + n_cwo * (n_pairs - 1 - g)
        pm[w:w + n_cwo] = g
    return pm


def _symmetric_slabs(n, width, seed, salt, spread):
    """[n][width][width] symmetric Gaussian slabs, N(0, 1/spread), decaying over n as the auxiliary spectrum does."""
    gen = _gen(seed, salt)
    b = torch.empty((n, width, width), dtype=torch.float64, device=DEV)
    decay = 0.5 / math.sqrt(spread) * torch.exp(-3.0 * torch.arange(n, dtype=torch.float64, device=DEV) / n)
    step = max(1, (1 << 26) // (width * width))
    for i in range(0, n, step):
        G = torch.randn((min(step, n - i), width, width), dtype=torch.float64, device=DEV, generator=gen)
        torch.add(G, G.transpose(1, 2), out=b[i:i + step])
        b[i:i + step] *= decay[i:i + step, None, None]
    return b


def _molecule(m, seed, salt=0):
    nb, npair, ncwo = m["n_bf"], m["n_pairs"], m["n_cwo"]
    rng = np.random.default_rng([seed, salt, 1])
    C, _ = np.linalg.qr(rng.standard_normal((nb, nb)))
    H = rng.standard_normal((nb, nb))
    H = np.triu(H) + np.triu(H, 1).T
    pm = _pair_map(npair, ncwo)
    strong = rng.uniform(0.9, 0.99, npair)
    occ = np.concatenate([strong, (1.0 - strong[pm[npair:]]) / ncwo])
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for k, v in (("C", C), ("H", H), ("occ", occ), ("pair_of", pm))}
    t["b"] = _symmetric_slabs(m["n_aux"], nb, seed, 17 * salt + 2, nb)
    return t


def _batch_mols(case):
    sizes = np.random.default_rng(case["sizes"]).integers(case["lo"], case["hi"] + 1, size=case["n_mol"])
    return [_mol(int(n), 3 * int(n), max(2, int(n) // 12), case["n_cwo"]) for n in sizes]


def _metric(case, seed):
    n = case["n_aux"]
    rng = np.random.default_rng([seed, 3])
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    w = np.geomspace(1.0, 1.0 / case["cond"], n)
    if case["negative"]:
        w[-case["negative"]:] = -1e-3 / case["cond"]
    G = (Q * w) @ Q.T
    return (G + G.T) / 2


def _three_centre(case, seed):
    gen = _gen(seed, 5)
    G = torch.randn((case["n_aux"], case["n_bf"], case["n_bf"]), dtype=torch.float64, device=DEV, generator=gen)
    return (G + G.transpose(1, 2)) * (0.5 / math.sqrt(case["n_bf"]))


def _orbital_inputs(case, seed):
    """Multipliers of an iteration under way: orbital energies on the diagonal, the residual asymmetry off it."""
    n, w, nb = case["n_mo"], case["n_omega"], case["n_bf"]
    rng = np.random.default_rng([seed, 7])
    eps = np.sort(rng.normal(0.0, 5.0, n))
    lam = 0.2 * rng.standard_normal((n, w))
    lam[np.arange(w), np.arange(w)] = eps[:w]
    C, _ = np.linalg.qr(rng.standard_normal((nb, n)))
    return lam, eps, np.ascontiguousarray(C)


def _on_problems(case, seed):
    """J, K and H_pp of many molecules: C^T b C of the recipe's b is a Gaussian symmetric block of the pairing space itself."""
    rng = np.random.default_rng(case["sizes"])
    val = np.random.default_rng([seed, 9])
    got = []
    for i in range(case["n_mol"]):
        nb = int(rng.integers(case["lo"], case["hi"] + 1))
        npair, ncwo = nb // 12, int(rng.integers(1, 7))
        w = npair * (1 + ncwo)
        bmo = _symmetric_slabs(3 * nb, w, seed, 31 * i + 11, nb)
        d = torch.diagonal(bmo, dim1=1, dim2=2)
        J = (d.T @ d).contiguous()
        K = (bmo * bmo).sum(0)
        Hpp = torch.from_numpy(val.standard_normal(w)).to(DEV)
        got.append((Hpp, J, K, torch.from_numpy(_pair_map(npair, ncwo)).to(DEV), npair, ncwo))
    return got


def _cold_rows(onset):
    P = torch.zeros((onset.rows, N_OUT), dtype=torch.float32)
    r = 0
    for npair, ncwo in onset.sizes:
        P[r:r + npair, 0] = 0.98
        P[r:r + npair, 1:1 + min(ncwo, 6)] = 0.02 / ncwo
        r += npair
    return P.to(DEV)


def _train_inputs(case, seed):
    """Standardised features, masks and targets, and the weights and Adam state of a training under way."""
    rows, gen = case["rows"], _gen(seed, 13)
    r = lambda *s: torch.randn(s, dtype=torch.float32, device=DEV, generator=gen)  # noqa: E731
    ncwo = torch.randint(1, 7, (rows, 1), device=DEV, generator=gen)
    M = (torch.arange(N_OUT, device=DEV)[None, :] <= ncwo).float()
    X = r(rows, N_IN)
    X[:, 3:33] *= M[:, 1:].repeat_interleave(5, 1)
    X[:, 33:] = M[:, 1:]
    strong = 0.9 + 0.09 * torch.rand((rows, 1), device=DEV, generator=gen)
    share = torch.rand((rows, N_OUT - 1), device=DEV, generator=gen) * M[:, 1:] + 1e-3 * M[:, 1:]
    T = torch.cat([strong, (1.0 - strong) * share / share.sum(1, keepdim=True)], 1)
    parts = []
    for i, o in ((N_IN, N_HID), (N_HID, N_HID), (N_HID, N_HID), (N_HID, N_OUT)):
        parts += [r(i * o) * math.sqrt(2.0 / (i + o)), 0.05 * r(o)]
    theta = torch.cat(parts)
    m, v = 1e-4 * r(theta.numel()), 1e-6 * (0.5 + torch.rand(theta.shape, device=DEV, generator=gen))
    return {"X": X.contiguous(), "M": M.contiguous(), "T": T.contiguous(), "theta": theta, "m": m, "v": v}


_contexts = {}


def _context(tune):
    """The handle a program keeps: one context per kind for the process."""
    if tune not in _contexts:
        _contexts[tune] = rif.Context(0)
        _contexts[tune].autotune(tune)
    return _contexts[tune]


# ---- the cases ---------------------------------------------------------------
def prepare(case, seed):
    what = case["what"]
    ctx = _context(case.get("tune", what == "prepare"))
    s = {"case": case, "ctx": ctx}
    if what in ("build", "direct"):
        prec = PREC[case["prec"]]
        s["in"] = _molecule(case, seed)
        s["out"] = ctx.outputs(case["n_bf"], case["n_aux"], case["n_pairs"], case["n_cwo"], case["n_bf"], prec, DEV, per_mo_ao=what == "build")
        s["split"] = ctx.presplit_b(s["in"]["b"], prec) if case["presplit"] else None
        if case["tune"]:
            run(s)
    elif what == "batch":
        mols = _batch_mols(case)
        prec = PREC[case["prec"]]
        shapes = [_shapes(m) for m in mols]
        # one array per output for the whole batch, each molecule's part starting 16-byte aligned
        s["out"] = {k: torch.zeros(sum(_even(math.prod(sh[k])) for sh in shapes), dtype=_out_type(k, prec), device=DEV) for k in OUT}
        at, items = dict.fromkeys(OUT, 0), []
        for i, (m, sh) in enumerate(zip(mols, shapes)):
            o = {}
            for k in OUT:
                n = math.prod(sh[k])
                o[k] = s["out"][k][at[k]:at[k] + n].view(sh[k])
                at[k] += _even(n)
            items.append((_molecule(m, seed, i), m["n_pairs"], m["n_cwo"], o))
        s["batch"] = ctx.batch(items, prec)
    elif what == "prepare":
        s["T"], s["G"] = _three_centre(case, seed), torch.from_numpy(_metric(case, seed)).to(DEV)
        s["b"] = torch.empty_like(s["T"])
        run(s)
    elif what == "orbital":
        s["lam"], s["eps"], s["C"] = (torch.from_numpy(x).to(DEV) for x in _orbital_inputs(case, seed))
        s["eps_out"] = torch.empty_like(s["eps"])
    elif what == "on":
        s["set"] = rif.OnSet(ctx, _on_problems(case, seed))
        s["P"] = _cold_rows(s["set"])
    elif what == "train":
        s.update(_train_inputs(case, seed))
        f, n = torch.float32, case["rows"]
        s["H"], s["dA"] = torch.empty((3, n, N_HID), dtype=f, device=DEV), torch.empty((2, n, N_HID), dtype=f, device=DEV)
        s["Z"], s["Pn"] = torch.empty((n, N_OUT), dtype=f, device=DEV), torch.empty((n, N_OUT), dtype=f, device=DEV)
        s["grad"], s["loss"], s["step"] = torch.zeros_like(s["theta"]), torch.zeros(1, dtype=torch.float64, device=DEV), 200
    else:
        s["in"] = _molecule(case, seed)
        s["gamma"] = torch.zeros(case["n_pairs"] * case["n_cwo"], dtype=torch.float64, device=DEV)
        s["out"] = ctx.outputs(case["n_bf"], case["n_aux"], case["n_pairs"], case["n_cwo"], case["n_bf"], rif.FP64, DEV, per_mo_ao=False)
    return s


def run(s):
    case, ctx, what = s["case"], s["ctx"], s["case"]["what"]
    if what in ("build", "direct"):
        t = s["in"]
        f = ctx.build if what == "build" else ctx.build_direct
        return f(t["b"], t["C"], t["H"], t["occ"], t["pair_of"], case["n_pairs"], case["n_cwo"], prec=PREC[case["prec"]], out=s["out"], b_split=s["split"])
    if what == "batch":
        s["batch"].run(True)
        return s["out"]
    if what == "prepare":
        return ctx.prepare_b(s["T"], s["G"], b=s["b"])
    if what == "orbital":
        eps = ctx.orbital_step(s["lam"], s["C"], case["n_omega"], eps_in=s["eps"], eps_out=s["eps_out"])
        return {"eps": eps, "C": s["C"]}
    if what == "on":
        ctx.on_warmstart(s["set"], s["P"])
        ctx.on_optimize(s["set"])
        return {"gamma": s["set"].gamma, "occ": s["set"].occ, "energy": s["set"].energy, "status": s["set"].status}
    if what == "train":
        s["step"] += 1
        ctx.mlp_forward(s["X"], s["M"], s["theta"], s["H"], s["Z"], s["Pn"])
        ctx.mlp_backward(s["X"], s["M"], s["T"], s["theta"], s["H"], s["Z"], s["dA"], s["grad"], s["loss"])
        ctx.adam(s["theta"], s["grad"], s["m"], s["v"], s["step"], 1e-3)
        return {k: s[k] for k in ("theta", "m", "v", "grad", "loss", "Z", "Pn")}
    t = s["in"]
    C, occ, gamma = t["C"].clone(), t["occ"].clone(), s["gamma"].clone()
    res, he, hg = ctx.optimize(t["b"], C, t["H"], occ, gamma, t["pair_of"], case["n_pairs"], case["n_cwo"], max_outer=1, max_inner=case["inner"],
                               tol_grad=1e-14, hist_len=case["inner"], out=s["out"])
    return {"energies": he, "grads": hg, "C": C, "occ": occ, "gamma": gamma, "inner": res["inner_total"]}


def _even(n):
    return n + n % 2


def _out_type(k, prec):
    return torch.float32 if prec != rif.FP64 and k in ("b_half", "b_mo", "Jn", "Kn") else torch.float64


def _shapes(m):
    nb, na, w = m["n_bf"], m["n_aux"], m["n_pairs"] * (1 + m["n_cwo"])
    return {"b_half": (w, na, nb), "b_mo": (na, w, w), "d": (na, w), "J": (w, w), "K": (w, w), "Jn": (w, nb, nb), "Kn": (w, nb, nb),
            "energy": (1,), "lam": (nb, w), "grad": (nb, nb)}


def _build_work(m, prec, what="build", presplit=False):
    """J^q, K^q, K_pq and b_mo are symmetric: half their products.  The Coulomb part of F^(q) c_q follows from b_half
    and d, the exchange part takes one product per (q, r) pair of K^r and c_q (build) or of b_mo and b_half (direct)."""
    nb, na, w = float(m["n_bf"]), float(m["n_aux"]), float(m["n_pairs"] * (1 + m["n_cwo"]))
    io = 8.0 if prec == "fp64" else 4.0
    b = 2.0 * PIECES[prec] if presplit and prec in PIECES else 4.0 if presplit else 8.0
    flops = 2 * na * nb * nb * w + na * nb * w * (w + 1) + 2 * na * w * (w + 1) + 4 * na * w * nb + 4 * nb * nb * w
    bytes_ = b * na * nb * nb + io * (w * na * nb + na * w * w) + 8 * (na * w + 2 * w * w + 4 * nb * nb)
    if what == "build":
        flops += 2 * na * w * nb * (nb + 1) + 2 * w * w * nb * nb
        bytes_ += 2 * io * w * nb * nb
    else:
        flops += 2 * na * w * w * nb
    return {"bytes": bytes_, "flops": flops}


def work(case):
    what = case["what"]
    if what in ("build", "direct"):
        return _build_work(case, case["prec"], what, case["presplit"])
    if what == "batch":
        each = [_build_work(m, case["prec"]) for m in _batch_mols(case)]
        return {k: sum(x[k] for x in each) for k in ("bytes", "flops")}
    if what == "prepare":
        nb, na = float(case["n_bf"]), float(case["n_aux"])
        return {"bytes": 8 * (1.5 * na * nb * nb + na * na), "flops": na ** 3 / 3 + na * na * nb * (nb + 1) / 2}
    if what == "orbital":
        n, nb = float(case["n_mo"]), float(case["n_bf"])
        return {"bytes": 8 * (n * case["n_omega"] + 2 * nb * n + 2 * n), "flops": 9 * n ** 3 + 2 * nb * n * n}
    if what == "on":
        rng = np.random.default_rng(case["sizes"])
        pairs = []
        for _ in range(case["n_mol"]):
            nb = int(rng.integers(case["lo"], case["hi"] + 1))
            pairs.append((nb // 12, int(rng.integers(1, 7))))
        ws = [p * (1 + c) for p, c in pairs]
        # about 24 iterations, one evaluation of every (p, q) term each
        return {"bytes": sum(8.0 * (2 * w * w + 4 * w) for w in ws), "flops": sum(24 * 30.0 * w * w for w in ws)}
    if what == "train":
        n, macs = float(case["rows"]), N_IN * N_HID + 2 * N_HID * N_HID + N_HID * N_OUT
        return {"bytes": 4 * n * (N_IN + 4 * N_OUT) + 4.0 * 8 * macs, "flops": 2 * n * (3 * macs - N_IN * N_HID)}
    one = _build_work(case, "fp64", "direct")
    n = float(case["n_bf"])
    return {"bytes": one["bytes"], "flops": case["inner"] * (one["flops"] + 11 * n ** 3)}


# ---- what plain torch gives in 64 bits ----------------------------------------
def _exact_build(t, m, what="build"):
    nb, na, npair, w = m["n_bf"], m["n_aux"], m["n_pairs"], m["n_pairs"] * (1 + m["n_cwo"])
    b, C, H, n = t["b"], t["C"], t["H"], t["occ"]
    Co = C[:, :w].contiguous()
    bh = (b.reshape(na * nb, nb) @ Co).reshape(na, nb, w).permute(2, 0, 1).contiguous()
    bmo = (bh.reshape(w * na, nb) @ Co).reshape(w, na, w).permute(1, 0, 2).contiguous()
    d = torch.diagonal(bmo, dim1=1, dim2=2).contiguous()
    J, K = d.T @ d, (bmo * bmo).sum(0)
    p = t["pair_of"].long()
    same = p[:, None] == p[None, :]
    weak = torch.arange(w, device=DEV) >= npair
    phi = torch.sqrt(n * (1 - n))
    nn = torch.outer(n, n)
    A = torch.where(same, torch.zeros_like(nn), 2 * nn)
    within = torch.where(weak[:, None] & weak[None, :], torch.sqrt(nn), -torch.sqrt(nn))
    within = torch.where(torch.eye(w, dtype=torch.bool, device=DEV), n[:, None].expand(w, w), within)
    B = torch.where(same, within, -nn - torch.outer(phi, phi))
    Hpp = ((H @ Co) * Co).sum(0)
    E = 2 * (n * Hpp).sum() + (A * J).sum() + (B * K).sum()
    out = {"b_half": bh, "b_mo": bmo, "d": d, "J": J, "K": K, "energy": E.reshape(1)}
    Y = (H @ Co) * n + torch.stack([(d @ A[q]) @ bh[q] for q in range(w)], 1)
    if what == "build":
        out["Jn"] = (d.T @ b.reshape(na, nb * nb)).reshape(w, nb, nb)
        out["Kn"] = torch.stack([bh[q].T @ bh[q] for q in range(w)])
        for r in range(w):
            Y += out["Kn"][r] @ (Co * B[:, r])
    else:
        out["Jn"] = out["Kn"] = None
        for r in range(w):
            Y += bh[r].T @ (bmo[:, r, :] * B[:, r])
    out["lam"] = C.T @ Y
    full = torch.zeros((nb, nb), dtype=torch.float64, device=DEV)
    full[:, :w] = out["lam"]
    out["grad"] = 4 * (full - full.T)
    return out


def _exact_prepare(case, seed):
    G = _metric(case, seed)
    n, alpha = G.shape[0], (1 + math.sqrt(17)) / 8
    delta = 2.0 ** -26 * np.abs(G).sum(1).max()
    A, L, perm, k = G.copy(), np.eye(n), np.arange(n), 0
    Dih = np.zeros((n, n))
    while k < n:
        akk, step, kp = abs(A[k, k]), 1, k
        col = np.abs(A[k + 1:, k])
        cmax = col.max() if col.size else 0.0
        if akk < alpha * cmax:
            im = k + 1 + int(np.argmax(col))
            row = np.abs(A[im, k:]).copy()
            row[im - k] = 0.0
            rmax = row.max()
            if akk * rmax < alpha * cmax * cmax:
                kp, step = im, 1 if abs(A[im, im]) >= alpha * rmax else 2
        kk = k + step - 1
        if kp != kk:
            A[[kk, kp], :] = A[[kp, kk], :]
            A[:, [kk, kp]] = A[:, [kp, kk]]
            L[[kk, kp], :k] = L[[kp, kk], :k]
            perm[[kk, kp]] = perm[[kp, kk]]
        E, W = A[k:k + step, k:k + step].copy(), A[k + step:, k:k + step].copy()
        if step == 2 or E[0, 0] != 0.0:
            L[k + step:, k:k + step] = W @ np.linalg.inv(E)
            A[k + step:, k + step:] -= L[k + step:, k:k + step] @ W.T
        w, Q = np.linalg.eigh(E)
        Dih[k:k + step, k:k + step] = (Q / np.sqrt(np.maximum(w, delta))) @ Q.T
        k += step
    T = _three_centre(case, seed)
    M = torch.from_numpy(Dih @ np.linalg.solve(L, np.eye(n))).to(DEV)
    return (M @ T[torch.from_numpy(perm).to(DEV)].reshape(n, -1)).reshape(T.shape)


def _exact_train(case, seed):
    s = {k: v.double() for k, v in _train_inputs(case, seed).items()}
    theta = s["theta"].clone().requires_grad_(True)
    x, at = s["X"], 0
    for i, o in ((N_IN, N_HID), (N_HID, N_HID), (N_HID, N_HID), (N_HID, N_OUT)):
        x = x @ theta[at:at + i * o].view(i, o) + theta[at + i * o:at + (i + 1) * o]
        at += (i + 1) * o
        x = torch.tanh(x) if o == N_HID else x
    P = torch.softmax(x.masked_fill(s["M"] == 0, -torch.inf), 1)
    loss = (s["M"] * (P - s["T"]) ** 2).sum() / case["rows"]
    g, = torch.autograd.grad(loss, theta)
    m, v = 0.9 * s["m"] + 0.1 * g, 0.999 * s["v"] + 0.001 * g * g
    new = s["theta"] - 1e-3 * (m / (1 - 0.9 ** 201)) / (torch.sqrt(v / (1 - 0.999 ** 201)) + 1e-8)
    return {"theta": new, "m": m, "v": v, "grad": g, "loss": loss.detach().reshape(1), "Z": x.detach(), "Pn": P.detach()}


def exact(case, seed):
    what = case["what"]
    if what in ("build", "direct"):
        return _exact_build(_molecule(case, seed), case, what)
    if what == "batch":
        parts = {k: [] for k in OUT}
        for i, m in enumerate(_batch_mols(case)):
            o = _exact_build(_molecule(m, seed, i), m)
            for k in OUT:
                x = o[k].reshape(-1)
                parts[k].append(torch.nn.functional.pad(x, (0, x.numel() % 2)))
        return {k: torch.cat(v) for k, v in parts.items()}
    if what == "prepare":
        return _exact_prepare(case, seed)
    if what == "orbital":
        lam, eps, _ = _orbital_inputs(case, seed)
        n, w = case["n_mo"], case["n_omega"]
        full = np.zeros((n, n))
        full[:, :w] = lam
        low = np.tril(full - full.T, -1)
        return {"eps": np.linalg.eigvalsh(low + low.T + np.diag(eps)), "C": None}  # C's columns are fixed up to their signs
    if what == "train":
        return _exact_train(case, seed)
    return None  # on, loop: the end of an iteration, which a tolerance or a step count ends
