"""What the speed of this framework is measured on: the calls that its users make, over the sizes they make
them at.

The kinds of call, each through the public binding (``paper_1107_5719_amd.rt3d``):

* ``fs``      one formal solution J_fs = Lambda S of a given source, with the emergent light of the top;
* ``step``    one operator-splitting step from a given J: formal solution, residual, inner Jacobi sweeps;
* ``lstar``   a new medium: its upload, the check, and the 27-point Lambda* operator;
* ``solve``   a new medium solved to convergence;
* ``batch``   many wavelengths on grids of different sizes solved to convergence together;
* ``adjoint`` the gradients of a loss on the emergent light through a converged solution.

The media are stratified atmospheres as in ``paper_1107_5719_amd.inputs`` (opacity falling by seven decades
over the column, log-normal noise), drawn on the GPU from the seed.  ``exact`` traces the lines with plain
torch in float64, from the geometry alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1107_5719_amd import rt3d

DEVICE = "cuda"


def _case(name, kind, nx, ny, nz, n_theta, n_phi, precision="fp64", eps=1e-2, tau=1e3, sweeps=30, accel="ng",
          tol=1e-8, members=1, bottom=0, i_top=0.0):
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "n_theta": n_theta, "n_phi": n_phi, "precision": precision,
         "eps": eps, "tau": tau, "sweeps": sweeps, "accel": accel, "tol": tol, "members": members,
         "bottom": bottom, "i_top": i_top}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a formal solution on the smallest grid in use (a parity-sized problem): launches and latency count
        _case("fs_17", "fs", 17, 17, 17, 8, 8),
        # the paper's smaller timing grid with 16 x 16 angles
        _case("fs_65", "fs", 65, 65, 65, 16, 16, eps=1e-4, tau=1e4),
        # the benchmark's grid
        _case("fs_129", "fs", 129, 129, 129, 16, 16, eps=1e-6),
        # the paper's larger timing grid in the FP32 form (single precision is what the paper timed first)
        _case("fs_slab_fp32", "fs", 129, 129, 193, 16, 16, precision="fp32"),
        # an uneven domain, irradiated from above and with the LTE-diffusion inner boundary
        _case("fs_ragged", "fs", 97, 41, 58, 8, 16, bottom=2, i_top=0.3),
        # one operator-splitting step: what an outer iteration repeats, on the smallest and the benchmark's grid
        _case("step_17", "step", 17, 17, 17, 8, 8),
        _case("step_129", "step", 129, 129, 129, 16, 16, eps=1e-6),
        # a new medium: Lambda* is built once for each
        _case("lstar_65", "lstar", 65, 65, 65, 16, 16, eps=1e-4, tau=1e4),
        # whole solves of a new medium: small with Ng acceleration, mid-size in the FP32 form with Anderson mixing
        _case("solve_17", "solve", 17, 17, 17, 8, 8),
        _case("solve_65_fp32", "solve", 65, 65, 65, 8, 8, precision="fp32", accel="anderson", sweeps=12, tol=1e-11),
        # wavelengths of one atmosphere, each on a grid of its own, solved together
        _case("batch_12", "batch", 97, 97, 97, 8, 8, accel="anderson", sweeps=4, tol=1e-9, members=12),
        # the backward pass of the differentiable solve
        _case("adjoint_65", "adjoint", 65, 65, 65, 8, 8, tol=1e-10),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fs", "fs", "step", "step", "lstar", "solve", "batch", "adjoint"])
    n_theta, n_phi = rng.choice([8, 16]), rng.choice([8, 16])
    hi = {"fs": 129, "step": 129, "lstar": 80, "solve": 80, "batch": 97, "adjoint": 65}[kind]
    nx, ny, nz = _size(rng, 12, hi), _size(rng, 12, hi), _size(rng, 12, hi)
    precision = rng.choice(["fp64", "fp64", "fp32"])
    bottom, i_top = rng.choice([0, 0, 1, 2]), rng.choice([0.0, 0.0, round(rng.uniform(0.05, 0.5), 3)])
    eps = 10.0 ** round(rng.uniform(-4.0, -1.0), 2)
    tau = 10.0 ** round(rng.uniform(2.0, 4.0), 2)
    sweeps, accel, tol, members = rng.choice([8, 12, 20, 30]), "ng", 1e-8, 1
    if kind == "solve":
        accel, tol, eps = rng.choice(["ng", "anderson"]), 1e-11 if precision == "fp32" else 1e-10, max(eps, 1e-3)
    elif kind == "batch":
        n_theta = n_phi = 8
        accel, eps, members = "anderson", max(eps, 1e-3), rng.randint(3, 10)
        tol = 1e-11 if precision == "fp32" else 1e-9
    elif kind == "adjoint":
        n_theta = n_phi = 8
        precision, tol, eps = "fp64", 1e-10, max(eps, 1e-3)
    return _case(None, kind, nx, ny, nz, n_theta, n_phi, precision, eps, tau, sweeps, accel, tol, members, bottom,
                 i_top)


# ---- inputs ---------------------------------------------------------------------------------------------------


def _medium(nx, ny, nz, eps, tau, gen):
    """chi, eps, B of a stratified atmosphere, and a J that the iteration would meet (falling to sqrt(eps) at the
    top)."""
    H = nz / (7.0 * math.log(10.0))
    z = torch.arange(nz, dtype=torch.float64, device=DEVICE) + 0.5
    prof = torch.exp(-z / H)
    prof = prof * (tau / prof.sum())

    def noise():
        return torch.randn((nz, ny, nx), generator=gen, dtype=torch.float64, device=DEVICE)

    chi = prof[:, None, None] * torch.exp(0.05 * noise())
    B = torch.full((nz, ny, nx), 1.0, dtype=torch.float64, device=DEVICE)
    B *= (1.5 - 0.5 * z / nz)[:, None, None]
    depth = torch.flip(torch.cumsum(torch.flip(prof, [0]), 0), [0])
    root = math.sqrt(eps)
    J = B * (root + (1.0 - root) * depth / (1.0 + depth))[:, None, None] * torch.exp(0.02 * noise())
    return chi, torch.full_like(chi, eps), B, J


def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _members(case, seed):
    """Grid, eps and tau of every wavelength of a batch: edges between a third of the case's and its own."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for m in range(case["members"]):
        f = (1.0, 0.67, 0.34)[m % 3]
        grid = {"nx": max(8, round(f * case["nx"])), "ny": max(8, round(f * case["ny"])),
                "nz": max(8, round(f * case["nz"])), "n_theta": case["n_theta"], "n_phi": case["n_phi"],
                "I_top": case["i_top"], "bottom_bc": case["bottom"]}
        eps = float(np.exp(rng.uniform(np.log(case["eps"]), np.log(0.1 + case["eps"]))))
        tau = float(np.exp(rng.uniform(np.log(0.01 * case["tau"]), np.log(case["tau"]))))
        out.append((grid, eps, tau))
    return out


def _accelerate(handle, case):
    if case["accel"] == "anderson":
        handle.set_anderson(8)
    else:
        handle.set_acceleration(3, 6)


def _precision(case):
    return rt3d.RT3D_FP32_SWEEP if case["precision"] == "fp32" else rt3d.RT3D_FP64


def prepare(case, seed):
    gen = _generator(seed)
    if case["kind"] == "batch":
        members = _members(case, seed)
        batch = rt3d.Batch([g for g, _, _ in members], precision=_precision(case))
        _accelerate(batch, case)
        media = [_medium(g["nx"], g["ny"], g["nz"], e, t, gen)[:3] for g, e, t in members]
        torch.cuda.synchronize()      # the batch runs on a stream of its own
        return {"case": case, "batch": batch, "media": media, "J": [torch.empty_like(m[0]) for m in media]}
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    s = rt3d.Solver(nx, ny, nz, case["n_theta"], case["n_phi"], case["i_top"], case["bottom"], _precision(case))
    chi, eps, B, J = _medium(nx, ny, nz, case["eps"], case["tau"], gen)
    out = {"case": case, "solver": s, "medium": (chi, eps, B), "J0": J, "out": torch.empty_like(chi)}
    if case["kind"] == "lstar":
        out["L"] = torch.empty((27, nz, ny, nx), dtype=torch.float64, device=DEVICE)
        return out
    s.set_medium(chi, eps, B)
    if case["kind"] == "fs":
        out["S"] = eps * B + (1.0 - eps) * J
    if case["kind"] in ("fs", "adjoint"):
        out["top"] = torch.empty((s.n_dir // 2, ny, nx), dtype=torch.float64, device=DEVICE)
    if case["kind"] == "step":
        s.build_lstar()
    if case["kind"] in ("solve", "adjoint"):
        _accelerate(s, case)
    if case["kind"] == "adjoint":
        s.solve(1e-11, 2000, case["sweeps"])
        out["g"] = torch.rand(out["top"].shape, generator=gen, dtype=torch.float64, device=DEVICE) - 0.3
        out["dchi"], out["deps"] = torch.empty_like(chi), torch.empty_like(chi)
    return out


# ---- one pass -------------------------------------------------------------------------------------------------


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        b = state["batch"]
        for m, medium in enumerate(state["media"]):
            b.set_medium(m, *medium)
        b.solve(case["tol"], 500, case["sweeps"])
        for m, J in enumerate(state["J"]):
            b.get_J(m, J)
        return {"J": state["J"]}
    s = state["solver"]
    if kind == "fs":
        s.formal_solution(state["S"], state["out"])
        s.emergent_top(state["top"])
        if case["precision"] == "fp32":
            # float32 sweeps carry float32 accuracy: a caller keeps their result in that type
            return {"J": state["out"].float(), "top": state["top"].float()}
        return {"J": state["out"], "top": state["top"]}
    if kind == "step":
        s.set_J(state["J0"])
        c = s.os_step(case["sweeps"])
        return {"J": s.get_J(state["out"]), "c": c}
    if kind == "lstar":
        s.set_medium(*state["medium"])
        s.build_lstar()
        return {"L": s.get_lstar(state["L"])}
    if kind == "solve":
        s.set_medium(*state["medium"])
        s.solve(case["tol"], 2000, case["sweeps"])
        return {"J": s.get_J(state["out"])}
    dchi, deps, *_ = s.adjoint(state["g"], case["tol"], 2000, case["sweeps"], dchi=state["dchi"], deps=state["deps"])
    return {"dchi": dchi, "deps": deps}


# ---- what a pass cannot do without ----------------------------------------------------------------------------


def _segments(n_theta, n_phi):
    """Mean segments that a line has in a voxel layer, times the directions: 1 + tan(theta) (|cos| + |sin|)."""
    mu, _ = np.polynomial.legendre.leggauss(n_theta)
    phi = 2.0 * math.pi * (np.arange(n_phi) + 0.5) / n_phi
    t = np.sqrt(1.0 - mu * mu) / np.abs(mu)
    return float((1.0 + t[:, None] * (np.abs(np.cos(phi)) + np.abs(np.sin(phi)))[None, :]).sum())


# Per line segment: an exponential (about 24 operations), shared by the two lines of an x-mirrored pair, and each
# line's intensity and deposit (7).
_FLOPS_SEGMENT = 19


def work(case):
    V = case["nx"] * case["ny"] * case["nz"]
    n_dir = case["n_theta"] * case["n_phi"]
    seg = _segments(case["n_theta"], case["n_phi"])
    top = 8 * (n_dir // 2) * case["nx"] * case["ny"]
    fs = {"bytes": 24 * V, "flops": V * seg * _FLOPS_SEGMENT}
    jac = {"bytes": (13 * (4 if case["precision"] == "fp32" else 8) + 32) * V, "flops": 54 * V}
    # Lambda*: every segment's exponential and self term, and about two neighbours reached from it
    lstar = {"bytes": (8 + 27 * 8) * V, "flops": V * seg * 60}
    M = case["sweeps"]
    if case["kind"] == "fs":
        return {"bytes": fs["bytes"] + top, "flops": fs["flops"]}
    if case["kind"] == "step":
        return {"bytes": fs["bytes"] + M * jac["bytes"] + 16 * V, "flops": fs["flops"] + M * jac["flops"]}
    if case["kind"] == "lstar":
        return {"bytes": lstar["bytes"] + 48 * V, "flops": lstar["flops"]}
    # whole solves: the outer steps that such media take
    steps = 20
    one = {k: fs[k] + M * jac[k] for k in fs}
    if case["kind"] == "batch":
        share = sum((1.0, 0.67, 0.34)[m % 3] ** 3 for m in range(case["members"]))
        return {k: share * (steps * one[k] + lstar[k]) for k in one}
    if case["kind"] == "adjoint":
        return {k: steps * one[k] + 3 * fs[k] for k in one}
    return {k: steps * one[k] + lstar[k] for k in one}


# ---- 64-bit references in plain torch -------------------------------------------------------------------------


def _crossings(nz, t, k):
    """Heights inside layer k where the line 1/2 + (z - nz) t crosses an integer."""
    if t == 0.0:
        return []
    a, b = sorted((0.5 + (k - nz) * t, 0.5 + (k + 1 - nz) * t))
    return [nz + (m - 0.5) / t for m in range(math.floor(a) + 1, math.ceil(b))]


def _layer(nz, mu, ox, oy, k):
    """(di, dj, length) of the pieces of the line through the centre of its top column, in travel order."""
    tx, ty = ox / mu, oy / mu
    z = sorted({float(k), float(k + 1), *_crossings(nz, tx, k), *_crossings(nz, ty, k)}, reverse=mu < 0)
    out = []
    for z0, z1 in zip(z, z[1:]):
        zm = 0.5 * (z0 + z1)
        out.append((math.floor(0.5 + (zm - nz) * tx), math.floor(0.5 + (zm - nz) * ty), abs(z1 - z0) / abs(mu)))
    return out


def _quads(case):
    """One direction of every four that are mirrored in x and y (phi in the first quadrant), with its weight and the
    directions' indices in the order of the flips (), (x), (y), (x, y)."""
    mu, w = np.polynomial.legendre.leggauss(case["n_theta"])
    n = case["n_phi"]
    for a in range(case["n_theta"]):
        s = math.sqrt(1.0 - mu[a] ** 2)
        for b in range(n // 4):
            phi = 2.0 * math.pi * (b + 0.5) / n
            dirs = [a * n + q for q in (b, n // 2 - 1 - b, n - 1 - b, n // 2 + b)]
            yield float(mu[a]), s * math.cos(phi), s * math.sin(phi), float(w[a]) / (2.0 * n), dirs


def _flips(x):
    """The four mirrored copies of [..., ny, nx] planes, stacked before the last two axes."""
    return torch.stack([x, x.flip(-1), x.flip(-2), x.flip((-1, -2))], dim=-3)


def _unflip(x):
    return x[..., 0, :, :], x[..., 1, :, :].flip(-1), x[..., 2, :, :].flip(-2), x[..., 3, :, :].flip((-1, -2))


def _exact_fs(case, chi, S, B):
    nz, ny, nx = chi.shape
    cf, sf, bf = _flips(chi), _flips(S), _flips(B[0])
    slope = _flips((B[0] - B[1]) / (0.5 * (chi[0] + chi[1])))
    J = torch.zeros_like(cf)
    top = torch.zeros((case["n_theta"] * case["n_phi"] // 2, ny, nx), dtype=torch.float64, device=chi.device)
    for mu, ox, oy, w, dirs in _quads(case):
        I = torch.full_like(cf[0], case["i_top"])
        order = range(nz - 1, -1, -1) if mu < 0 else range(nz)
        for n, k in enumerate(order):
            segs = _layer(nz, mu, ox, oy, k)
            if n == 0 and mu > 0:
                at = (-segs[0][1], -segs[0][0])
                I = torch.zeros_like(I)
                if case["bottom"] != 1:
                    I = torch.roll(bf + mu * slope if case["bottom"] == 2 else bf, at, (-2, -1))
            for di, dj, length in segs:
                # voxel (i + di, j + dj) of the line whose top column is (i, j)
                c, s = torch.roll(cf[k], (-dj, -di), (-2, -1)), torch.roll(sf[k], (-dj, -di), (-2, -1))
                tau = c * length
                d = (I - s) * torch.expm1(-tau)
                I = I + d
                J[k] += torch.roll(s * tau - d, (dj, di), (-2, -1)) * (w * abs(mu))
        if mu > 0:
            for d, plane in zip(dirs, _unflip(I)):
                top[d - top.shape[0]] = plane
    return sum(_unflip(J)) / chi, top


def _exact_lstar(case, chi):
    """Lambda*_{v,o}: derivative of J_v by S at v's neighbour o = 9 (dk + 1) + 3 (dj + 1) + di + 1."""
    nz, ny, nx = chi.shape
    cf = _flips(chi)
    L = torch.zeros((27, nz, 4, ny, nx), dtype=torch.float64, device=chi.device)

    def near(m, n):
        m %= n
        return m if m < 2 else (-1 if m == n - 1 else None)

    for mu, ox, oy, w, _ in _quads(case):
        wmu = w * abs(mu)
        layers = [_layer(nz, mu, ox, oy, k) for k in range(nz)]
        for k in range(nz):
            up = k + 1 if mu < 0 else k - 1
            before = [(p, up) for p in layers[up]] if 0 <= up < nz else []
            line = before + [(p, k) for p in layers[k]]
            for q in range(len(before), len(line)):
                (ai, aj, length), _ = line[q]
                tau = cf[k] * length
                em1 = torch.expm1(-tau)
                small = tau * tau * (0.5 - tau / 6 * (1 - tau / 4 * (1 - tau / 5 * (1 - tau / 6))))
                L[13, k] += wmu * torch.where(tau < 1e-2, small, tau + em1)
                T = torch.ones_like(tau)
                for (bi, bj, lb), kb in reversed(line[:q]):
                    di, dj = bi - ai, bj - aj
                    tb = torch.roll(cf[kb], (-dj, -di), (-2, -1)) * lb
                    oi, oj = near(di, nx), near(dj, ny)
                    if oi is not None and oj is not None:
                        L[9 * (kb - k + 1) + 3 * (oj + 1) + oi + 1, k] += wmu * em1 * torch.expm1(-tb) * T
                    T = T * torch.exp(-tb)
    L = L / cf
    out = torch.zeros((27, nz, ny, nx), dtype=torch.float64, device=chi.device)
    for o in range(27):
        dk, dj, di = o // 9, (o // 3) % 3, o % 3
        for f, plane in enumerate(_unflip(L[o])):
            # a flip mirrors the neighbour's offset too
            out[9 * dk + 3 * (2 - dj if f >= 2 else dj) + (2 - di if f % 2 else di)] += plane
    return out


def _exact_step(case, chi, eps, B, J):
    r = _exact_fs(case, chi, eps * B + (1.0 - eps) * J, B)[0] - J
    L = _exact_lstar(case, chi)
    diag = 1.0 - L[13] * (1.0 - eps)
    dJ = torch.zeros_like(r)
    for _ in range(case["sweeps"]):
        x = torch.nn.functional.pad(((1.0 - eps) * dJ).permute(1, 2, 0), (1, 1)).permute(2, 0, 1)
        acc = r.clone()
        for o in range(27):
            if o != 13:
                dk, dj, di = o // 9 - 1, (o // 3) % 3 - 1, o % 3 - 1
                acc += L[o] * torch.roll(x, (-dj, -di), (1, 2))[1 + dk:1 + dk + chi.shape[0]]
        dJ = acc / diag
    return J + dJ


def _exact_cost(case):
    """Segments that the reference traces one after another (times the walk back, for Lambda*)."""
    mean = _segments(case["n_theta"], case["n_phi"]) / 4.0
    return mean * case["nz"], mean * case["nz"] * 1.5 * mean / (case["n_theta"] * case["n_phi"] / 4)


def exact(case, seed):
    if case["kind"] not in ("fs", "step", "lstar"):
        return None
    lines, walks = _exact_cost(case)
    if case["kind"] != "fs" and walks > 60000:
        return None
    chi, eps, B, J = _medium(case["nx"], case["ny"], case["nz"], case["eps"], case["tau"], _generator(seed))
    if case["kind"] == "fs":
        Jfs, top = _exact_fs(case, chi, eps * B + (1.0 - eps) * J, B)
        return {"J": Jfs, "top": top}
    if case["kind"] == "lstar":
        return {"L": _exact_lstar(case, chi)}
    return {"J": _exact_step(case, chi, eps, B, J), "c": None}
