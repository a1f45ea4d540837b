"""Timing cases of the framework's public entry points.

Networks, cells and request streams come from the seeded generators of synth:
the 12-, 200- and 500-species networks of the benchmark, and reduced networks
of any size between (the first species the larger one's reactions reach from
the atoms, with every reaction among them).  Matrices and abundances are drawn
here.  Horizons are
1e3..1e6 yr on the 12-species network and 1e3..1e5 yr on the larger ones (the
last decade to the benchmark's 1e6 yr adds under a tenth of the steps); rtol
1e-6 and atol 1e-20 throughout, the benchmark's.
"""
import math

import numpy as np
import torch

import paper_2511_10558_amd as ab
import synth

DEV = "cuda:0"
F64 = torch.float64
_NETS: dict = {}


def listed():
    return [
        # the coefficients of a whole batch before its solve: the benchmark's 4096 cells of 500 species
        {"name": "rates_500sp_4096", "kind": "rates", "species": 500, "cells": 4096},
        # the right-hand side on its own (an external integrator's call), the benchmark's batch
        {"name": "rhs_500sp_4096", "kind": "rhs", "species": 500, "cells": 4096},
        # dense Newton matrices for a caller's own linear algebra
        {"name": "newton_matrix_200sp_192", "kind": "newton_matrix", "species": 200, "cells": 192},
        # batched factorisation of Newton matrices at the largest order used
        {"name": "lu_factor_500x256", "kind": "lu_factor", "species": 500, "cells": 256},
        # batched solves with given factors
        {"name": "lu_solve_500x256", "kind": "lu_solve", "species": 500, "cells": 256},
        # the smallest solve: one cell of the 12-species network, latency alone
        {"name": "solve_12sp_1", "kind": "solve", "species": 12, "cells": 1, "t_end_yr": 1e6,
         "lu_reuse": 0.0, "precision": "fp64", "method": "bdf"},
        # an ordinary batch of the middle network
        {"name": "solve_200sp_250", "kind": "solve", "species": 200, "cells": 250, "t_end_yr": 1e5,
         "lu_reuse": 0.3, "precision": "fp64", "method": "bdf"},
        # the benchmark's network and factorisation policy, more cells than compute units
        {"name": "solve_500sp_512", "kind": "solve", "species": 500, "cells": 512, "t_end_yr": 1e5,
         "lu_reuse": 0.3, "precision": "fp64", "method": "bdf"},
        # the FP32-factorisation form
        {"name": "solve_500sp_96_fp32lu", "kind": "solve", "species": 500, "cells": 96,
         "t_end_yr": 1e4, "lu_reuse": 0.3, "precision": "fp32_lu", "method": "bdf"},
        # the ESDIRK integrator on a network of no round size
        {"name": "esdirk_131sp_67", "kind": "solve", "species": 131, "cells": 67, "t_end_yr": 1e5,
         "lu_reuse": 0.0, "precision": "fp64", "method": "esdirk5"},
        # a training step: forward with tape, gradients of log alpha, x0 and the physical parameters
        {"name": "grad_200sp_64", "kind": "grad", "species": 200, "cells": 64, "t_end_yr": 1e4},
        # a server taking requests of 1..64 cells with mixed horizons
        {"name": "serve_200sp_12req", "kind": "serve", "species": 200, "requests": 12,
         "max_cells": 64, "slots": 256, "lu_reuse": 0.3, "precision": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_net(rng, most):
    """A size between 12 species and `most`: the benchmark's three, or any."""
    s = rng.choice([12, 200, 500, 0, 0, 0])
    return _log_int(rng, 24, min(most, 490)) if s == 0 or s > most else s


def draw(rng):
    kind = rng.choice(["rates", "rhs", "newton_matrix", "lu_factor", "lu_solve", "solve", "solve", "solve", "grad",
                       "serve"])
    if kind in ("rates", "rhs"):
        s = _draw_net(rng, 500)
        return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 4096)}
    if kind in ("newton_matrix", "lu_factor", "lu_solve"):
        s = _draw_net(rng, 500)
        return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 256)}
    if kind == "serve":
        s = _draw_net(rng, 200)
        return {"kind": kind, "species": s, "requests": rng.randrange(1, 13),
                "max_cells": _log_int(rng, 4, 64), "slots": rng.randrange(96, 257), "lu_reuse": rng.choice([0.0, 0.3]),
                "precision": "fp64"}
    if kind == "grad":
        s = _draw_net(rng, 200)
        return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 64),
                "t_end_yr": 10.0 ** rng.uniform(3.0, 4.0)}
    form = rng.choice(["fp64", "fp64", "fp64", "fp32_lu", "esdirk5"])
    if form == "fp64":
        s = _draw_net(rng, 500)
        return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 512),
                "t_end_yr": 10.0 ** rng.uniform(3.0, 6.0 if s == 12 else 5.0), "lu_reuse": rng.choice([0.0, 0.3]),
                "precision": "fp64", "method": "bdf"}
    if form == "fp32_lu":
        s = _draw_net(rng, 500)
        return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 96),
                "t_end_yr": 10.0 ** rng.uniform(3.0, 4.0), "lu_reuse": 0.3, "precision": "fp32_lu", "method": "bdf"}
    s = _draw_net(rng, 200)
    return {"kind": kind, "species": s, "cells": _log_int(rng, 1, 67),
            "t_end_yr": 10.0 ** rng.uniform(3.0, 5.0), "lu_reuse": 0.0, "precision": "fp64", "method": "esdirk5"}


def _arrays(species):
    """The synthetic network of this many species."""
    for name, size in (("small", 12), ("net200", 200), ("net500", 500)):
        if species <= size:
            full = synth.network_for_config(name)
            break
    if species == full.n_species:
        return full
    order = [full.index(a) for a in ("e-", "H", "He", "C", "N", "O", "S")]
    sides = np.concatenate([full.reactants, full.products], axis=1)
    for i in sides.ravel():
        if i >= 0 and i not in order:
            order.append(int(i))
    keep = sorted(order[:species])          # ascending, so rows of species stay ascending
    new = np.full(full.n_species + 1, -1, np.int32)
    new[keep] = np.arange(len(keep))        # new[-1] stays -1: no species
    inside = ((sides < 0) | (new[sides] >= 0)).all(axis=1)
    return synth.Network(f"{full.name}-{len(keep)}", [full.species[i] for i in keep], full.comp[keep],
                         full.charge[keep], full.rtype[inside], new[full.reactants[inside]],
                         new[full.products[inside]], full.alpha[inside], full.beta[inside], full.gamma[inside],
                         full.albedo)


def _net(case):
    """The case's network (arrays and handle), loaded once as a program would."""
    key = case["species"]
    if key not in _NETS:
        net = _arrays(key)
        _NETS[key] = (net, ab.Network.from_text(net.to_text()))
    return _NETS[key]


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=F64, device=DEV)


def _cells(net, n, seed, t_end_yr):
    c = synth.sample_cells(net, n, seed=seed, t_end_yr=t_end_yr)
    return [_t(v) for v in (c.T, c.n_H, c.A_V, c.zeta, c.G0, c.x0, c.t_end)]


def _state_inputs(net, n, seed):
    """Coefficients, abundances and c = h / gamma of cells on their way: every
    species above 1e-14, c from the first steps to late ones."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.exp(math.log(1e-14) * torch.rand((n, net.n_species), generator=g, dtype=F64, device=DEV))
    c = torch.exp(math.log(1e3) + math.log(1e7) * torch.rand((n,), generator=g, dtype=F64, device=DEV))
    return _rates64(net, *_cells(net, n, seed, 1e5)[:5]), x, c


def _rates64(net, T, nH, Av, zeta, G0):
    al, be, ga = (_t(v)[None, :] for v in (net.alpha, net.beta, net.gamma))
    t = torch.tensor(np.asarray(net.rtype), device=DEV)[None, :]
    T, nH, Av, zeta, G0 = (v[:, None] for v in (T, nH, Av, zeta, G0))
    two = al * (T / 300.0) ** be * torch.exp(-ga / T) * nH
    photo = al * G0 * torch.exp(-ga * Av)
    return torch.where(t == synth.TWO_BODY, two, torch.where(t == synth.COSMIC_RAY, al * zeta, photo)).contiguous()


def _nu(net):
    """The stoichiometric matrix [S, R]."""
    nu = np.zeros((net.n_species, net.n_reactions))
    for col, sign in ((net.reactants, -1.0), (net.products, 1.0)):
        for j in range(col.shape[1]):
            m = col[:, j] >= 0
            np.add.at(nu, (col[m, j], np.nonzero(m)[0]), sign)
    return _t(nu)


def _reactants(net):
    re = torch.tensor(np.asarray(net.reactants, dtype=np.int64), device=DEV)
    return re[:, 0], re[:, 1]


def _newton64(net, k, x, c):
    """I - c J(x) per cell: J = nu . d rate / dx."""
    a, b = _reactants(net)
    one = b < 0
    bb = torch.where(one, a, b)
    nu, S, R = _nu(net), net.n_species, net.n_reactions
    r = torch.arange(R, device=DEV)
    out = torch.empty((x.shape[0], S, S), dtype=F64, device=DEV)
    eye = torch.eye(S, dtype=F64, device=DEV)
    for i in range(x.shape[0]):
        d = torch.zeros((R, S), dtype=F64, device=DEV)
        xb = torch.where(one, torch.ones_like(x[i, bb]), x[i, bb])
        d[r, a] = k[i] * xb
        two = ~one
        # A + A has both derivatives in one entry
        d[r[two], b[two]] += k[i][two] * x[i, a[two]]
        out[i] = eye - c[i] * (nu @ d)
    return out


def prepare(case, seed):
    net, g = _net(case)
    kind, st = case["kind"], {"case": case, "net": net, "g": g}
    if kind == "rates":
        st["args"] = _cells(net, case["cells"], seed, 1e5)[:5]
    elif kind == "rhs":
        st["k"], st["x"], _ = _state_inputs(net, case["cells"], seed)
    elif kind == "newton_matrix":
        st["k"], st["x"], st["c"] = _state_inputs(net, case["cells"], seed)
    elif kind == "lu_factor":
        st["A"] = _newton64(net, *_state_inputs(net, case["cells"], seed))
    elif kind == "lu_solve":
        A = _newton64(net, *_state_inputs(net, case["cells"], seed))
        st["LU"], st["perm"] = _lu64(A)
        gen = torch.Generator(device=DEV).manual_seed(seed)
        st["b"] = torch.randn(A.shape[:2], generator=gen, dtype=F64, device=DEV)
    elif kind == "solve":
        st["args"] = _cells(net, case["cells"], seed, case["t_end_yr"])
        st["options"] = ab.make_options(rtol=1e-6, atol=1e-20, lu_reuse=case["lu_reuse"], precision=case["precision"],
                                        method=case["method"])
    elif kind == "grad":
        a = _cells(net, case["cells"], seed, case["t_end_yr"])
        st["args"] = [v.requires_grad_(True) for v in a[:6]] + [a[6]]
        st["log_alpha"] = _t(np.log(net.alpha)).requires_grad_(True)
        gen = torch.Generator(device=DEV).manual_seed(seed)
        st["w"] = torch.randn(a[5].shape, generator=gen, dtype=F64, device=DEV)
        st["options"] = ab.make_options(rtol=1e-6, atol=1e-20)
    else:
        st["server"] = ab.Server(g, max_slots=case["slots"], lu_reuse=case["lu_reuse"], precision=case["precision"])
        # the stream's sizes are the case's, its conditions and horizons the seed's
        sizes = [r.cells.n for r in synth.request_stream(net, case["requests"], 5, 1.0, case["max_cells"])]
        rng = np.random.default_rng(seed)
        st["requests"] = [synth.sample_cells(net, n, int(rng.integers(2**31)), 10.0 ** rng.uniform(3.0, 5.0))
                          for n in sizes]
    return st


def run(state):
    kind, g = state["case"]["kind"], state["g"]
    if kind == "rates":
        return ab.rates(g, *state["args"])
    if kind == "rhs":
        return ab.rhs(g, state["k"], state["x"])
    if kind == "newton_matrix":
        return ab.newton_matrix(g, state["k"], state["x"], state["c"])
    if kind == "lu_factor":
        return ab.lu_factor(state["A"])
    if kind == "lu_solve":
        return ab.lu_solve(state["LU"], state["perm"], state["b"])
    if kind == "solve":
        return ab.solve(g, *state["args"], options=state["options"])
    if kind == "grad":
        a = state["args"]
        x, status = ab.solve_diff(g, *a, state["log_alpha"], options=state["options"])
        grads = torch.autograd.grad((state["w"] * x).sum(), [state["log_alpha"], *a[:4], a[5]])
        return [x.detach(), status, *grads]
    srv, live, out = state["server"], {}, [None] * len(state["requests"])
    for i, c in enumerate(state["requests"]):
        live[srv.submit(c.T, c.n_H, c.A_V, c.zeta, c.G0, c.x0, c.t_end)] = i
    while live:
        for d in srv.poll(timeout_ms=1000):
            out[live.pop(d["id"])] = (d["x"], d["status"])
    return out


def _counts(case):
    """Factorisations and Newton iterations a cell takes, about, by what the
    integrators need on these networks at these tolerances."""
    if case["species"] == 12:
        return 120.0, 1400.0
    if case["kind"] == "solve" and case["method"] == "esdirk5":
        return 100.0, 1600.0
    return (70.0, 800.0) if case["species"] < 350 else (75.0, 1200.0)


def work(case):
    s, kind = case["species"], case["kind"]
    r = _net(case)[0].n_reactions
    if kind == "serve":
        # mean of floor(exp(U[0, ln(max + 1)))) cells a request
        n = case["requests"] * max(1.0, case["max_cells"] / math.log(case["max_cells"] + 1.0) - 0.5)
    else:
        n = case["cells"]
    if kind == "rates":
        return {"bytes": 8.0 * (n * (5 + r) + 3 * r), "flops": 40.0 * n * r}
    if kind == "rhs":
        return {"bytes": 8.0 * n * (2 * s + r), "flops": n * r * 11.0}
    if kind == "newton_matrix":
        return {"bytes": 8.0 * n * (s * s + s + r + 1), "flops": n * (r * 18.0 + s * s)}
    if kind == "lu_factor":
        return {"bytes": n * (16.0 * s * s + 4.0 * s), "flops": n * 2.0 / 3.0 * s ** 3}
    if kind == "lu_solve":
        return {"bytes": n * (8.0 * s * s + 20.0 * s), "flops": n * 2.0 * s * s}
    lu, it = _counts(case)
    flops = n * (lu * 2.0 / 3.0 * s ** 3 + it * (2.0 * s * s + 11.0 * r))
    byts = 8.0 * n * (2 * s + 6) + 24.0 * r
    if kind == "grad":
        # the sweep: one transposed factorisation and solve per accepted step, and the gradients
        flops += n * 300.0 * (2.0 / 3.0 * s ** 3 + 2.0 * s * s + 30.0 * r)
        byts += 8.0 * (n * (2 * s + 5) + r)
    return {"bytes": byts, "flops": flops}


def exact(case, seed):
    """In plain torch, 64 bits; the integrations have no such value (their
    result is defined by the step control, not by a formula)."""
    kind = case["kind"]
    if kind in ("solve", "grad", "serve"):
        return None
    net, n = _net(case)[0], case["cells"]
    if kind == "rates":
        return _rates64(net, *_cells(net, n, seed, 1e5)[:5])
    k, x, c = _state_inputs(net, n, seed)
    if kind == "rhs":
        a, b = _reactants(net)
        nu, f = _nu(net), torch.empty_like(x)
        for i in range(0, n, 64):
            xa, xb = x[i:i + 64][:, a], torch.where(b < 0, torch.ones_like(k[i:i + 64]), x[i:i + 64][:, b])
            f[i:i + 64] = (k[i:i + 64] * xa * xb) @ nu.T.contiguous()
        return f
    A = _newton64(net, k, x, c)
    if kind == "newton_matrix":
        return A
    if kind == "lu_solve":
        LU, perm = _lu64(A)
        gen = torch.Generator(device=DEV).manual_seed(seed)
        b = torch.randn(A.shape[:2], generator=gen, dtype=F64, device=DEV)
        y = b.gather(1, perm.long())
        for i in range(1, y.shape[1]):
            y[:, i] -= (LU[:, i, :i] * y[:, :i]).sum(dim=1)
        for i in range(y.shape[1] - 1, -1, -1):
            y[:, i] = (y[:, i] - (LU[:, i, i + 1:] * y[:, i + 1:]).sum(dim=1)) / LU[:, i, i]
        return y
    return [_lu64(A)[0], None, None]


def _lu64(A):
    """L and U of P A and the rows' order, with the pivots that lu_factor
    documents: per 16 columns the diagonal's while no multiplier exceeds 4, else
    partial pivoting."""
    A, n = A.clone(), A.shape[1]
    perm = torch.arange(n, dtype=torch.int32, device=DEV).repeat(A.shape[0], 1)
    every = torch.arange(A.shape[0], device=DEV)
    for c0 in range(0, n, 16):
        c1 = min(c0 + 16, n)
        P = A[:, c0:, c0:c1].clone()
        for j in range(c1 - c0):
            P[:, j + 1:, j] /= P[:, j, j, None]
            P[:, j + 1:, j + 1:] -= P[:, j + 1:, j, None] * P[:, j, None, j + 1:]
        ok = ((torch.tril(P, -1).abs() <= 4.0).all(dim=(1, 2)) & torch.isfinite(P).all(dim=(1, 2)))
        bad = every[~ok]
        if bad.numel():
            Q = A[bad, c0:, :].clone()      # whole rows: exchanges move them
            m = torch.arange(bad.numel(), device=DEV)
            for j in range(c1 - c0):
                cj = c0 + j
                p = Q[:, j:, cj].abs().argmax(dim=1) + j
                top, low = Q[:, j].clone(), Q[m, p].clone()
                Q[m, p], Q[:, j] = top, low
                top, low = perm[bad, cj].clone(), perm[bad, c0 + p].clone()
                perm[bad, c0 + p], perm[bad, cj] = top, low
                Q[:, j + 1:, cj] /= Q[:, j, cj, None]
                Q[:, j + 1:, cj + 1:c1] -= Q[:, j + 1:, cj, None] * Q[:, j, None, cj + 1:c1]
            A[bad, c0:, :] = Q
            P[bad] = Q[:, :, c0:c1]
        A[:, c0:, c0:c1] = P
        if c1 < n:
            w = c1 - c0
            U = A[:, c0:c1, c1:].clone()
            for j in range(1, w):
                U[:, j] -= (P[:, j, :j, None] * U[:, :j]).sum(dim=1)
            A[:, c0:c1, c1:] = U
            A[:, c1:, c1:] -= torch.bmm(P[:, w:, :w].contiguous(), U)
    return A, perm
