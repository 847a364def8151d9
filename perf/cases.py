"""The work that programs built on this library have it do, as cases that can be timed.

Most cases are one batched sign solve of a whole synthetic system (synth.water,
the systems of the tests and of bench.py) through `Solver`: from the 64-molecule
box of the parity tests, where launches and latency count, to the 4,096-molecule
cube at r_c 0.9 nm, in the four precisions and on the routes that the options
offer. Beside them: the chemical-potential search, and one training step of the
spectral-bound network.

A solve returns the block-sparse D (and W where it is asked for), the molecules'
electron counts, band energies, iteration counts and status. The block
pattern belongs to the case; the values of K and S come from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import synth
from paper_2104_08245_amd import Solver, _lib as L, learned, mlp_adam, mlp_loss_grad

BS = 6
DEV = "cuda:0"

# The routes by name: keyword arguments of Solver beside the precision.
ROUTES = {
    # Solver's own defaults: the iteration on A_J = S^-1 K - mu I, FP64 factor
    "default": {},
    # the default of bench.py for FP16 / BF16: symmetric iteration, FP64 factor applied in FP32
    "sym": dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32),
    # the same with submatrices combined by the cubic criterion
    "combine": dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32, combine=True),
    # learned spectral bounds on the symmetric iteration
    "learned": dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32, bounds=L.BOUNDS_LEARNED),
    # the paper's own inverse: coupled Newton-Schulz in the 16-bit type
    "coupled": dict(inverse=L.INV_COUPLED_NS),
}


def _solve(name, system, nmol, r_c, prec, route, mu=0.0, w=False, stream="side", entry="batch"):
    """stream: "side" is a stream of the caller's own (the batch replays as one
    graph), "default" is torch's default stream (direct launches)."""
    return dict(name=name, kind="solve", system=system, nmol=nmol, r_c=r_c, prec=prec, route=route,
                mu=mu, w=w, stream=stream, entry=entry)


def listed():
    return [
        # the smallest whole call: the 64-molecule box (150 to 222 rows a
        # submatrix), as an MD program on a small cell calls it at every step
        _solve("box64-fp16", "cube", 64, 0.6, "fp16", "sym"),
        # the same box with Solver's defaults (FP64) on the default stream
        _solve("box64-fp64", "cube", 64, 0.6, "fp64", "default", stream="default"),
        # the plain FP64 method on ordinary submatrices (516 to 708 rows): the
        # reference solve against which mixed runs are checked
        _solve("cube512-fp64", "cube", 512, 0.9, "fp64", "default"),
        # the FP32 path on the same kind of system, a ragged molecule count
        _solve("cube777-fp32", "cube", 777, 0.9, "fp32", "default", stream="default"),
        # production: the route and submatrix sizes of bench.py, a batch that
        # fills the GPU many times over
        _solve("cube4096-fp16", "cube", 4096, 0.9, "fp16", "sym"),
        # BF16 with learned bounds, as on the frames of a trajectory
        _solve("cube1501-bf16-learned", "cube", 1501, 0.9, "bf16", "learned"),
        # FP16 with Solver's default route and the energy-weighted density
        # matrix for the forces
        _solve("cube1000-fp16-w", "cube", 1000, 0.9, "fp16", "default", w=True),
        # uneven submatrices (about 330 to 1,520 rows): the two-density slab
        _solve("slab2048-fp16", "slab", 2048, 1.2, "fp16", "sym"),
        # combined submatrices: fewer and larger, several molecules each
        _solve("cube2000-fp16-combine", "cube", 2000, 0.9, "fp16", "combine"),
        # the paper's own route to the inverse
        _solve("cube600-fp16-coupled", "cube", 600, 0.9, "fp16", "coupled"),
        # the chemical-potential search: the first midpoint lies in a band,
        # where the iteration uses all its slots, later ones in the gap
        dict(name="bisect216-fp16", kind="bisect", nmol=216, r_c=0.7, prec="fp16", route="sym"),
        # one training step of the spectral-bound network at learned.train's batch
        dict(name="mlp-step-256", kind="train", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "cube", "cube", "cube", "slab", "combine", "coupled", "bisect", "train"])
    if kind == "train":
        return dict(kind="train", batch=_log_int(rng, 33, 1024))
    if kind == "bisect":
        return dict(kind="bisect", nmol=rng.randint(64, 216), r_c=round(rng.uniform(0.5, 0.6), 3),
                    prec=rng.choice(["fp16", "bf16"]), route="sym")
    if kind == "box":
        nmol = _log_int(rng, 20, 220)
        half = 0.49 * (nmol / synth.water.DENSITY) ** (1 / 3)
        prec = rng.choice(["fp64", "fp32", "fp16", "fp16", "bf16"])
        route = "default" if prec in ("fp64", "fp32") else rng.choice(["default", "sym", "sym"])
        c = _solve("", "cube", nmol, round(min(rng.uniform(0.42, 0.65), half), 3), prec, route,
                   mu=rng.choice([0.0, 0.1, -0.1]), stream=rng.choice(["side", "default"]),
                   entry=rng.choice(["batch", "batch", "noalloc"]))
    elif kind == "cube":
        prec = rng.choice(["fp64", "fp32", "fp16", "fp16", "bf16"])
        top = {"fp64": 512, "fp32": 777, "fp16": 4096, "bf16": 4096}[prec]
        route = "default" if prec in ("fp64", "fp32") else rng.choice(["default", "sym", "sym", "learned"])
        c = _solve("", "cube", _log_int(rng, 200, top if route != "default" else min(top, 1000)),
                   round(rng.uniform(0.68, 0.89), 3), prec, route, mu=rng.choice([0.0, 0.1, -0.1]),
                   w=route == "default" and rng.random() < 0.3, stream=rng.choice(["side", "side", "default"]))
    elif kind == "slab":
        c = _solve("", "slab", 2 * rng.randint(600, 1000), round(rng.uniform(0.9, 1.07), 3),
                   rng.choice(["fp16", "bf16"]), "sym")
    elif kind == "combine":
        c = _solve("", "cube", _log_int(rng, 200, 2000), round(rng.uniform(0.68, 0.89), 3),
                   rng.choice(["fp16", "bf16"]), "combine")
    else:
        c = _solve("", "cube", _log_int(rng, 150, 600), round(rng.uniform(0.68, 0.89), 3),
                   rng.choice(["fp16", "bf16"]), "coupled")
    del c["name"]
    return c


# --------------------------------------------------------------------- inputs
def _system(case, seed):
    """The molecules of a case stand where the generator's own streams put
    them, whatever the seed: the block pattern belongs to the case, as it
    stays from one step of a program to the next. Basis positions and onsite
    energies, so every value of K and S, come from the seed."""
    nmol, half = case["nmol"], case["nmol"] // 2
    place = synth.water.streams(1000 + nmol)[0]
    if case.get("system", "cube") == "slab":
        # the default slab's box with its lateral area scaled to the molecule count
        side = 8.0 * math.sqrt(nmol / 16384)
        box = np.array([side, side, synth.water.SLAB_BOX[2]])
        z = synth.water.SLAB_DENSE_Z
        dense = synth.water.rsa_region(place, half, box, np.zeros(3), np.array([side, side, z]), None)
        dilute = synth.water.rsa_region(place, half, box, np.array([0.0, 0.0, z]), box, dense)
        centres = np.concatenate([dense, dilute])
    else:
        box = synth.water.cubic_box(nmol)
        centres = synth.water.rsa_region(place, nmol, box, np.zeros(3), box, None)
    _, jitter, onsite, sample = synth.water.streams(seed)
    return synth.water.build_system(centres, box, case["r_c"], jitter, onsite, sample)


def _network(seed):
    """Parameters and feature norms of the spectral-bound network, of the size
    and spread of trained ones: hidden layers as learned.train starts them, an
    output layer that predicts extremes near 0.7 of the Gershgorin box."""
    rng = np.random.default_rng(seed)
    th = learned.init_params(rng)
    th[-130:-2] *= 0.02
    th[-2:] = 0.7
    mean = np.array([6.4, 0.0, 1.0, -1.2, 1.2, 2.0, 4.0, -5.0, 5.0, -5.0, 5.0, 40.0])
    std = np.array([0.1, 0.2, 0.2, 0.2, 0.2, 0.5, 1.0, 1.0, 1.0, 1.0, 1.0, 8.0])
    t = lambda a: torch.tensor(np.ascontiguousarray(a, np.float32), device=DEV)  # noqa: E731
    return t(th), t(np.concatenate([mean, std])), mean, std


def _training_set(case, seed):
    """A mini-batch in the middle of a training run: raw features and targets
    (normalised extremes), Adam's moments of the size that they then have."""
    params, norm, mean, std = _network(seed)
    rng = np.random.default_rng(seed + 1)
    x = mean + std * rng.standard_normal((case["batch"], L.MLP_NFEAT))
    y = rng.uniform(0.45, 0.95, (case["batch"], 2))
    t = lambda a: torch.tensor(np.ascontiguousarray(a, np.float32), device=DEV)  # noqa: E731
    return dict(params=params, norm=norm, x=t(x), y=t(y),
                m=t(1e-3 * rng.standard_normal(L.MLP_NPARAM)),
                v=t(1e-6 * (0.5 + rng.random(L.MLP_NPARAM))),
                grad=torch.zeros(L.MLP_NPARAM, device=DEV), loss=torch.zeros(1, device=DEV), t=500)


def prepare(case, seed):
    if case["kind"] == "train":
        return dict(case=case, **_training_set(case, seed))
    kw = dict(ROUTES[case["route"]])
    keep = None
    if case["route"] == "learned":
        keep = _network(7)   # one trained network serves every input
        kw.update(d_mlp=keep[0].data_ptr(), d_mlp_norm=keep[1].data_ptr())
    if case.get("entry") == "noalloc":
        kw.update(ws_bytes=L.NOALLOC_WS_BYTES)
    sv = Solver(_system(case, seed), prec=case["prec"], device=DEV, **kw)
    if case.get("w"):
        sv.want_w()
    stream = torch.cuda.Stream() if case.get("stream", "side") == "side" else None
    words = sv.stats.view(torch.int32).reshape(sv.nb, -1)      # nolsm_mol_stats of each molecule
    reals = sv.stats.view(torch.float64).reshape(sv.nb, -1)
    out = dict(D=sv.D, N=reals[:, 4], E=reals[:, 5], iters=words[:, 0], status=words[:, 3])
    if case.get("w"):
        out["W"] = sv.Wcols
    return dict(case=case, sv=sv, stream=stream, keep=keep, out=out)


def run(state):
    case = state["case"]
    if case["kind"] == "train":
        s = state
        mlp_loss_grad(s["params"], s["norm"], s["x"], s["y"], s["grad"], s["loss"])
        mlp_adam(s["params"], s["grad"], s["m"], s["v"], s["t"], lr=1e-3)
        s["t"] += 1
        return dict(params=s["params"], m=s["m"], v=s["v"], grad=s["grad"], loss=s["loss"])
    sv = state["sv"]
    if case["kind"] == "bisect":
        # 4 occupied orbitals a molecule; midpoints -1 (in the lower band), then 0
        mu, count, steps, _ = sv.mu_bisect(-3.0, 1.0, 4.0 * case["nmol"], stream=state["stream"], allow_noconv=True)
        return dict(state["out"], mu=mu, count=count, steps=steps)
    if case["entry"] == "noalloc":
        sv.run_noalloc(mu=case["mu"], stream=state["stream"])
    else:
        sv.run(mu=case["mu"], stream=state["stream"])
    return state["out"]


# ----------------------------------------------------------- unavoidable work
def _sizes(case):
    """[(molecules, rows of a submatrix)] from the densities of the system."""
    ball = 4.0 / 3.0 * math.pi * case["r_c"] ** 3
    rows = lambda density: BS * (1.0 + ball * density)  # noqa: E731
    if case.get("system") == "slab":
        return [(case["nmol"] / 2, 0.85 * rows(synth.water.DENSITY)), (case["nmol"] / 2, rows(11.0))]
    return [(case["nmol"], min(BS * case["nmol"], rows(synth.water.DENSITY)))]


def work(case):
    """K and S read once, D (and W) written once; the products of the sign
    iteration at the iteration counts these systems take, in the form that the
    route runs (n^2 (n + 1) for a symmetric product, else 2 n^3), the factor of
    S, its application, and the n x 6 products of the finishing steps."""
    if case["kind"] == "train":
        p = L.MLP_NPARAM
        return {"bytes": 4.0 * (7 * p + 14 * case["batch"]), "flops": 6.0 * p * case["batch"]}
    solves = 2 if case["kind"] == "bisect" else 1
    iters = {"fp64": 16, "fp32": 14}.get(case["prec"], 13)
    if case["kind"] == "bisect":
        iters = 26   # mean of the slots used in a band (40) and in the gap
    sym = case["route"] in ("sym", "combine", "learned")
    nbytes = flops = 0.0
    for count, n in _sizes(case):
        blocks = n / BS
        nbytes += count * blocks * 36 * 8 * (4 if case.get("w") else 3)
        f = (2 * iters + 1) * (n * n * (n + 1) if sym else 2 * n ** 3)
        if case["route"] == "coupled":
            f += (3 * 9 + 2) * 2 * n ** 3
        else:
            f += n ** 3 / 3 + (n ** 3 if sym else 2 * n ** 3)
        if case["prec"] in ("fp16", "bf16"):
            f += 9 * 12 * n * n
        # combining saves some of this work; what it cannot do without is not known beforehand
        flops += count * f * (0.85 if case["route"] == "combine" else 1.0)
    return {"bytes": nbytes, "flops": flops * solves}


# ------------------------------------------------------------ 64-bit reference
def _exact_train(case, seed):
    s = _training_set(case, seed)
    d = {k: s[k].double() for k in ("params", "norm", "x", "y", "m", "v")}
    p = d["params"].clone().requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = torch.split(p, [64 * 12, 64, 64 * 64, 64, 2 * 64, 2])
    x = (d["x"] - d["norm"][:12]) / d["norm"][12:]
    silu = torch.nn.functional.silu
    h = silu(x @ w1.reshape(64, 12).t() + b1)
    h = silu(h @ w2.reshape(64, 64).t() + b2)
    e = h @ w3.reshape(2, 64).t() + b3 - d["y"]
    loss = (torch.where(e < 0, 4.0, 1.0) * e * e).mean()
    g, = torch.autograd.grad(loss, p)
    m = 0.9 * d["m"] + 0.1 * g
    v = 0.999 * d["v"] + 0.001 * g * g
    t = s["t"]
    new = d["params"] - 1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return dict(params=new, m=m, v=v, grad=g, loss=loss.detach().reshape(1))


def _padded(block, idx, real):
    """Dense submatrices from blocks: idx[b, i, j] is the stored block or -1;
    identity on the padding rows."""
    b, m, _ = idx.shape
    out = block[idx.clamp(min=0)] * (idx >= 0)[..., None, None]
    out = out.permute(0, 1, 3, 2, 4).reshape(b, m * BS, m * BS)
    pad = (~real).repeat_interleave(BS, 1).double()
    return out + torch.diag_embed(pad)


def exact(case, seed):
    """T_J(D) = (I - sign(S^-1 K - mu I)) S^-1 / 2 of every submatrix in 64 bits."""
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["route"] == "combine":
        return None   # another truncation: defined by the library's own groups
    s = _system(case, seed)
    mu = case.get("mu", 0.0)   # anywhere in the gap: the search ends there too
    nb = s.K.nb
    cols = torch.tensor(s.K.col_idx.astype(np.int64), device=DEV)
    ptr = torch.tensor(s.K.row_ptr.astype(np.int64), device=DEV)
    deg = ptr[1:] - ptr[:-1]
    rows = torch.repeat_interleave(torch.arange(nb, device=DEV), deg)
    keys = rows * nb + cols   # increasing: block-CSR order
    K = torch.tensor(s.K.val, device=DEV)
    S = torch.tensor(s.S.val, device=DEV)
    D = torch.zeros_like(K)
    want_w = bool(case.get("w"))
    W = torch.zeros_like(K) if want_w else None
    N = torch.zeros(nb, dtype=torch.float64, device=DEV)
    E = torch.zeros(nb, dtype=torch.float64, device=DEV)
    order = torch.argsort(deg).tolist()
    degs = deg.tolist()
    at = 0
    while at < nb:
        step = max(1, int(3e7 // (degs[order[min(nb - 1, at + 64)]] * BS) ** 2))
        js = torch.tensor(order[at:at + step], device=DEV)
        at += len(js)
        m = int(deg[js].max())
        slot = torch.arange(m, device=DEV)[None, :]
        real = slot < deg[js][:, None]
        entry = (ptr[js][:, None] + slot).clamp(max=len(cols) - 1)
        mol = torch.where(real, cols[entry], torch.full_like(entry, -1))
        key = mol[:, :, None] * nb + mol[:, None, :]
        idx = torch.searchsorted(keys, key.reshape(-1)).clamp(max=len(keys) - 1).reshape(key.shape)
        idx = torch.where((keys[idx] == key) & real[:, :, None] & real[:, None, :], idx, torch.full_like(idx, -1))
        TS, TK = _padded(S, idx, real), _padded(K, idx, real)
        own = (mol == js[:, None]).double()
        Ecol = torch.zeros(len(js), m, BS, BS, dtype=torch.float64, device=DEV)
        Ecol += own[:, :, None, None] * torch.eye(BS, dtype=torch.float64, device=DEV)
        Ecol = Ecol.reshape(len(js), m * BS, BS)
        # S^-1/2 by the coupled iteration (products only), then the sign of
        # S^-1/2 K S^-1/2 - mu I, whose D is the same
        c = 1.0 / TS.abs().sum(2).amax(1)[:, None, None]
        eye = torch.eye(m * BS, dtype=torch.float64, device=DEV)
        Y, Z = c * TS, eye.repeat(len(js), 1, 1)
        for _ in range(60):
            R = eye - torch.bmm(Z, Y)
            Y, Z = Y + 0.5 * torch.bmm(Y, R), Z + 0.5 * torch.bmm(R, Z)
            if float(R.square().sum((1, 2)).amax()) < 1e-14:
                break   # the step just taken squares this residual
        Z = c.sqrt() * 0.5 * (Z + Z.transpose(1, 2))
        A = torch.bmm(torch.bmm(Z, TK), Z)
        A = 0.5 * (A + A.transpose(1, 2)) - mu * eye * real.repeat_interleave(BS, 1).double()[:, :, None]
        y = torch.bmm(Z, Ecol)
        X = A / A.abs().sum(2).amax(1)[:, None, None]
        for _ in range(60):
            X2 = torch.bmm(X, X)
            err = float((X2 - eye).square().sum((1, 2)).amax())
            X = 1.5 * X - 0.5 * torch.bmm(X, X2)
            if err < 1e-14:
                break
        half_d = 0.5 * (y - torch.bmm(X, y))
        col = torch.bmm(Z, half_d)
        put = torch.where(real, mol * nb + js[:, None], torch.zeros_like(mol))
        where = torch.searchsorted(keys, put.reshape(-1)).clamp(max=len(keys) - 1)
        blocks = col.reshape(len(js) * m, BS, BS)
        flat = real.reshape(-1)
        D[where[flat]] = blocks[flat]
        if want_w:
            t = torch.bmm(A, half_d) + mu * half_d
            t = 0.5 * (t - torch.bmm(X, t))
            wc = torch.bmm(Z, t).reshape(len(js) * m, BS, BS)
            # W comes as column blocks: those of molecule J are row J's entries
            W[entry.reshape(-1)[flat]] = wc[flat]
        pick = own.argmax(1)
        rowS = TS.reshape(len(js), m, BS, -1)[torch.arange(len(js), device=DEV), pick]
        rowK = TK.reshape(len(js), m, BS, -1)[torch.arange(len(js), device=DEV), pick]
        N[js] = torch.einsum("bcr,brc->b", rowS, col)
        E[js] = torch.einsum("bcr,brc->b", rowK, col)
    out = dict(D=D.reshape(-1), N=N, E=E, iters=None, status=None)
    if want_w:
        out["W"] = W.reshape(-1)
    if case["kind"] == "bisect":
        out.update(mu=None, count=float(N.sum()), steps=None)
    return out
