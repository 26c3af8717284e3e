"""The workloads this library is timed on: block operators and their inverse,
block-local solves, the coupled operator of a box mesh, and whole
multigrid-preconditioned solves, each through the Python binding.

A case is a dict of plain values.  ``listed`` gives the fixed ones, ``draw``
another one of the same ranges, ``prepare`` what a program holds before the
call (device vectors in the plan's layout, the plan, its inverse, a solver),
``run`` one pass, ``work`` the bytes and operations a pass cannot do without,
and ``exact`` the outputs in 64 bits from plain torch and numpy.

Kinds:
  blocks    v = A u (volume operator) and x = D^{-1} b (cell block) on a batch
            of independent blocks of one degree
  mixed     the same two calls on a batch of several degrees, one launch each
  factors   the same two calls on blocks given by their own 1D factors
  solve     block-local iterative refinement of D x = b to 1e-10, from x = 0
  operator  v = A u with the coupled SIPG operator of a uniform box mesh
  mgsolve   A x = b on a box mesh by CG with one V-cycle per iteration
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2609_04534_amd import tpfdm

PENALTY = 2.0
DTYPES = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
CODES = {"f64": tpfdm.F64, "f32": tpfdm.F32}


def listed():
    return [
        # the smallest call: 512 cells of degree 2, where launches are all there is
        {"name": "blocks_p2_512_f64", "kind": "blocks", "degree": 2, "blocks": 512, "dtype": "f64"},
        # the headline batch: 64^3 affine cells of degree 3
        {"name": "blocks_p3_262144_f64", "kind": "blocks", "degree": 3, "blocks": 262144, "dtype": "f64"},
        # high degree with vectors stored in half precision
        {"name": "blocks_p7_32768_f16", "kind": "blocks", "degree": 7, "blocks": 32768, "dtype": "f16"},
        # a ragged mix of degrees in one batch, as an adaptive code has it
        {"name": "mixed_p237_20000_f32", "kind": "mixed", "blocks": 20000, "dtype": "f32"},
        # blocks with their own per-direction factors (no shared reference pair)
        {"name": "factors_p3_20011_f64", "kind": "factors", "degree": 3, "blocks": 20011, "dtype": "f64"},
        # block-local solves in mixed precision, the binding's default inner type
        {"name": "solve_p7_32768_f32", "kind": "solve", "degree": 7, "blocks": 32768, "inner": "f32"},
        # the coupled operator on the largest uniform cube (134 M unknowns)
        {"name": "operator_p3_128cube_f64", "kind": "operator", "degree": 3, "cells": "128x128x128",
         "dtype": "f64", "basis": "lagrange"},
        # ... at high degree
        {"name": "operator_p7_48cube_f64", "kind": "operator", "degree": 7, "cells": "48x48x48",
         "dtype": "f64", "basis": "lagrange"},
        # ... in the Hermite-type basis and FP32, on a box of odd counts
        {"name": "operator_p3_33x47x50_f32_hermite", "kind": "operator", "degree": 3, "cells": "33x47x50",
         "dtype": "f32", "basis": "hermite"},
        # whole solves: an ordinary mesh in FP64 under the preconditioned stopping rule
        {"name": "mgsolve_p3_64cube_f64", "kind": "mgsolve", "degree": 3, "cells": "64x64x64", "inner": "f64",
         "rule": "preconditioned"},
        # ... and two request classes of the serving mix (FP32 levels, residual rule)
        {"name": "mgsolve_p2_16cube_f32", "kind": "mgsolve", "degree": 2, "cells": "16x16x16", "inner": "f32",
         "rule": "residual"},
        {"name": "mgsolve_p7_24cube_f32", "kind": "mgsolve", "degree": 7, "cells": "24x24x24", "inner": "f32",
         "rule": "residual"},
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))

    kind = rng.choice(["blocks", "blocks", "mixed", "factors", "solve", "operator", "operator", "operator",
                       "mgsolve", "mgsolve"])
    p = rng.randint(1, 7)
    n3 = (p + 1) ** 3
    if kind == "blocks":
        return {"kind": kind, "degree": p, "blocks": spread(200, 4e7 / n3),
                "dtype": rng.choice(["f64", "f64", "f32", "f16", "bf16"])}
    if kind == "mixed":
        return {"kind": kind, "blocks": spread(300, 60000), "dtype": rng.choice(["f64", "f32"])}
    if kind == "factors":
        return {"kind": kind, "degree": p, "blocks": spread(100, min(40000, 4e6 / n3)),
                "dtype": rng.choice(["f64", "f32"])}
    if kind == "solve":
        return {"kind": kind, "degree": p, "blocks": spread(200, 2e7 / n3), "inner": rng.choice(["f64", "f32"])}
    if kind == "operator":
        side = float(np.exp(rng.uniform(np.log(5.0), np.log((4e7 / n3) ** (1 / 3)))))
        cells = "x".join(str(max(2, int(round(side * rng.uniform(0.75, 1.33))))) for _ in range(3))
        return {"kind": kind, "degree": p, "cells": cells, "dtype": rng.choice(["f64", "f32"]),
                "basis": rng.choice(["lagrange", "lagrange", "hermite"]) if p >= 3 else "lagrange"}
    # every mesh whose odd part the coarsest level solves directly
    sides = [m for m in (8, 12, 16, 24, 32, 48, 64) if m ** 3 * n3 <= 8_000_000]
    m = rng.choice(sides)
    cells = [m, m, m]
    if rng.random() < 0.4 and m & (m - 1) == 0:   # a box: one direction half as long
        cells[rng.randrange(3)] = m // 2
    return {"kind": "mgsolve", "degree": p, "cells": "x".join(map(str, cells)), "inner": rng.choice(["f64", "f32"]),
            "rule": rng.choice(["residual", "preconditioned"])}


# ---------------------------------------------------------------- inputs
def _cells(case):
    return tuple(int(c) for c in case["cells"].split("x"))


def _mesh_h(case):
    cells = _cells(case)
    return (1.0 / max(cells),) * 3   # cubes: the longest side of the box has length 1


def _mixed_counts(case):
    c = np.random.default_rng(case["blocks"]).multinomial(case["blocks"], [1 / 3] * 3)
    return list(zip((2, 3, 7), (int(v) for v in c)))


def _uniform(gen, shape, lo, hi, dtype=torch.float64):
    return torch.empty(shape, dtype=torch.float64, device="cuda").uniform_(lo, hi, generator=gen).to(dtype)


def _groups(case):
    """(degree, blocks) of every group of the case's plan."""
    if case["kind"] == "mixed":
        return _mixed_counts(case)
    if case["kind"] in ("operator", "mgsolve"):
        return [(case["degree"], int(np.prod(_cells(case))))]
    return [(case["degree"], case["blocks"])]


def _inputs(case, seed):
    """Edge lengths (or factors) per group and the canonical vectors u, b."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, groups = case["kind"], _groups(case)
    dtype = DTYPES[case.get("dtype", "f64")]
    out = {"h": [], "M": [], "P": []}
    for p, nb in groups:
        if kind in ("operator", "mgsolve"):
            continue
        h = _uniform(gen, (nb, 3), 0.5, 4.0 if p == 7 and kind != "mixed" else 2.0)
        out["h"].append(h)
        if kind == "factors":
            # the cell's pair, scaled per block and direction by its coefficients
            # and with a symmetric positive part of its own
            M, _, A = _reference(p)
            n = p + 1
            cm, cp = _uniform(gen, (nb, 3, 1, 1), 0.5, 2.0), _uniform(gen, (nb, 3, 1, 1), 0.5, 2.0)
            w, v = _uniform(gen, (nb, 3, n, 1), -1, 1), _uniform(gen, (nb, 3, n, 1), -1, 1)
            hh = h[:, :, None, None]
            out["M"].append(hh * (cm * _dev(M) + 0.1 / n * w * w.transpose(2, 3)))
            out["P"].append((cp * _dev(A) + v * v.transpose(2, 3)) / hh)
    ndof = sum(nb * (p + 1) ** 3 for p, nb in groups)
    out["u"] = _uniform(gen, (ndof,), -1, 1, dtype) if kind not in ("solve", "mgsolve") else None
    out["b"] = _uniform(gen, (ndof,), -1, 1, dtype) if kind != "operator" else None
    return out


def _packed(plan, v):
    """A canonical vector in the plan's layout (padding lanes zero)."""
    out = torch.zeros(plan.vector_elems, dtype=v.dtype, device="cuda")
    plan.pack(v, out)
    return out


def prepare(case, seed):
    kind = case["kind"]
    data = _inputs(case, seed)
    if kind in ("operator", "mgsolve"):
        basis = tpfdm.BASIS_HERMITE if case.get("basis") == "hermite" else tpfdm.BASIS_LAGRANGE
        plan = tpfdm.Plan.mesh(case["degree"] + 1, _cells(case), _mesh_h(case), penalty_C=PENALTY, basis=basis)
    else:
        specs = []
        for i, (p, _) in enumerate(_groups(case)):
            B = tpfdm.default_layout_B(p + 1)
            if kind == "factors":
                specs.append(tpfdm.GroupSpec(p + 1, B, None, M=data["M"][i], P=data["P"][i]))
            else:
                specs.append(tpfdm.GroupSpec(p + 1, B, data["h"][i]))
        plan = tpfdm.Plan(specs, penalty_C=PENALTY, persistent=kind == "mixed")
    state = {"kind": kind}
    if kind == "mgsolve":
        plan.setup_inverse(tpfdm.OP_CELL)
        inner = CODES[case["inner"]]
        state["solver"] = tpfdm.PCG(plan)
        state["solver"].set_multigrid(tpfdm.MG(plan, storage=inner))
        pre = case["rule"] == "preconditioned"
        state["solver"].set_norm(tpfdm.PCG_PRECONDITIONED if pre else tpfdm.PCG_RESIDUAL)
        state["inner"], state["rtol"] = inner, 1e-10 if pre else 1e-8
    elif kind != "operator":
        plan.setup_inverse(tpfdm.OP_CELL)
        state["inner"] = CODES.get(case.get("inner"))
    for name in ("u", "b"):
        if data[name] is not None:
            state[name] = _packed(plan, data[name])
    like = state["u"] if "u" in state else state["b"]
    state["v"], state["x"] = (torch.zeros_like(like) if name in state else None for name in ("u", "b"))
    state["plan"] = plan
    return state


def run(state):
    kind, plan = state["kind"], state["plan"]
    if kind == "operator":
        plan.apply(state["u"], state["v"], tpfdm.OP_SIPG)
        return state["v"]
    if kind == "mgsolve":
        state["solver"].solve(state["b"], state["x"], x_is_zero=True, inner=state["inner"], rtol=state["rtol"])
        return state["x"]
    if kind == "solve":
        state["x"].zero_()
        plan.solve(state["b"], state["x"], inner=state["inner"], rtol=1e-10)
        return state["x"]
    plan.apply(state["u"], state["v"], tpfdm.OP_NEUMANN)
    plan.apply_inverse(state["b"], state["x"])
    return [state["v"], state["x"]]


def work(case):
    kind = case["kind"]
    if kind in ("operator", "mgsolve"):
        p, nc = _groups(case)[0]
        n = p + 1
        nd = nc * n ** 3
        row = nc * (14 * n ** 4 + 24 * n * n * (n + 1))       # volume and face terms of A u
        inv = nc * 12 * n ** 4
        if kind == "operator":
            return {"bytes": 2 * nd * BYTES[case["dtype"]], "flops": row}
        # one iteration: the finest level's six updates (u, b read, u written; the
        # first from zero), residual and transfers, the levels below at 1/7 of
        # it, and eleven FP64 vectors of CG; iterations as measured per degree
        its = {1: 7, 2: 7, 3: 9}.get(p, 14)
        s = BYTES[case["inner"]]
        level = nd * s * (2 + 5 * 3 + 2 + 2)
        return {"bytes": its * (level * 8 / 7 + 11 * 8 * nd),
                "flops": its * ((6 * row + 6 * inv) * 8 / 7 + row + 12 * nd)}
    by = fl = 0
    for p, nb in _groups(case):
        n, s = p + 1, BYTES[case.get("dtype", "f64")]
        apply, inverse = 14 * n ** 4 + 2 * n ** 3, 12 * n ** 4 + n ** 3
        if kind == "solve":    # b read, x read and written; one correction
            by += nb * (3 * 8 * n ** 3 + 24)
            fl += nb * (apply + inverse)
        else:
            own = 8 * (3 * 2 * n * n + 3 * (n * n + n)) if kind == "factors" else 48
            by += nb * (4 * n ** 3 * s + own)
            fl += nb * (apply + inverse)
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------- the same in 64 bits
def _dev(a):
    return torch.as_tensor(a, dtype=torch.float64, device="cuda")


def _gauss_lobatto(points):
    inner = np.polynomial.legendre.Legendre.basis(points - 1).deriv().roots()
    return np.concatenate(([0.0], (1 + np.sort(np.real(inner))) / 2, [1.0]))


def _basis(p, basis="lagrange"):
    """The 1D basis on [0, 1] as polynomials."""
    poly = np.polynomial.Polynomial

    def lagrange(x, i):
        out = poly([1.0])
        for j in range(len(x)):
            if j != i:
                out = out * poly([-x[j], 1.0]) / (x[i] - x[j])
        return out

    if basis == "lagrange":
        x = _gauss_lobatto(p + 1)
        return [lagrange(x, i) for i in range(p + 1)]
    t, s = poly([0.0, 1.0]), poly([1.0, -1.0])
    x = _gauss_lobatto(p - 1)[1:-1]
    return ([s * s * (1 + 2 * t), t * s * s] + [lagrange(x, i) * t * t * s * s for i in range(len(x))]
            + [t * t * (t - 1), t * t * (3 - 2 * t)])


def _reference(p, basis="lagrange"):
    """Mass, stiffness and penalized cell operator of the 1D basis on [0, 1]."""
    f = _basis(p, basis)
    x, w = np.polynomial.legendre.leggauss(p + 3)
    x, w = (1 + x) / 2, w / 2
    V = np.array([q(x) for q in f])
    D = np.array([q.deriv()(x) for q in f])
    M, K = V * w @ V.T, D * w @ D.T
    e, g = _ends(p, basis)
    s = PENALTY * p * (p + 1)
    A = K + s * (np.outer(e[0], e[0]) + np.outer(e[1], e[1]))
    for side, sign in ((0, 0.5), (1, -0.5)):
        A = A + sign * (np.outer(e[side], g[side]) + np.outer(g[side], e[side]))
    return M, K, A


def _ends(p, basis):
    f = _basis(p, basis)
    return ([np.array([q(t) for q in f]) for t in (0.0, 1.0)],
            [np.array([q.deriv()(t) for q in f]) for t in (0.0, 1.0)])


def _mesh_1d(p, m, h, basis):
    """Mass and SIPG matrix of a line of m cells of length h."""
    M, K, _ = _reference(p, basis)
    e, g = _ends(p, basis)
    n, s = p + 1, PENALTY * p * (p + 1)
    S, Mg = np.kron(np.eye(m), K), np.kron(np.eye(m), M)
    for face in range(m + 1):
        j, a = np.zeros(m * n), np.zeros(m * n)   # jump and average of the normal derivative
        w = 0.5 if 0 < face < m else 1.0
        if face > 0:
            j[(face - 1) * n:face * n], a[(face - 1) * n:face * n] = e[1], w * g[1]
        if face < m:
            j[face * n:(face + 1) * n], a[face * n:(face + 1) * n] = -e[0], w * g[0]
        S += s * np.outer(j, j) - np.outer(j, a) - np.outer(a, j)
    return h * Mg, S / h


def _along(X, Y, Z, v):
    """(X (x) Y (x) Z) v for a tensor v of shape (x, y, z)."""
    v = torch.tensordot(v, _dev(Z), dims=([2], [1]))
    v = torch.tensordot(v, _dev(Y), dims=([1], [1])).transpose(1, 2)
    return torch.tensordot(_dev(X), v, dims=([1], [0]))


def _to_grid(case, v):
    (mx, my, mz), n = _cells(case), case["degree"] + 1
    v = v.reshape(mx, my, mz, n, n, n).permute(0, 3, 1, 4, 2, 5)
    return v.reshape(mx * n, my * n, mz * n)


def _from_grid(case, v):
    (mx, my, mz), n = _cells(case), case["degree"] + 1
    return v.reshape(mx, n, my, n, mz, n).permute(0, 2, 4, 1, 3, 5).reshape(-1)


def _blocked(groups, parts):
    """Canonical (blocks, n^3) arrays in the default layout of each group."""
    out = []
    for (p, nb), v in zip(groups, parts):
        B = 64 if p <= 3 else 1
        t = torch.zeros((nb + B - 1) // B * B, (p + 1) ** 3, dtype=torch.float64, device="cuda")
        t[:nb] = v.reshape(nb, -1)
        out.append(t.reshape(-1, B, (p + 1) ** 3).transpose(1, 2).reshape(-1))
    return torch.cat(out)


def _per_block(F, v, axis):
    """Contracts index `axis` (1..3) of v (blocks, n, n, n) with each block's F (blocks, n, n)."""
    w = v.movedim(axis, 1)
    n = v.shape[1]
    return torch.matmul(F, w.reshape(-1, n, n * n)).reshape(w.shape).movedim(1, axis)


def _kron_sum(M, P, u):
    out = 0
    for a in range(3):
        t = u
        for d in range(3):
            t = _per_block((P if d == a else M)[:, d].contiguous(), t, d + 1)
        out = out + t
    return out


def _kron_solve(M, P, b):
    """D^{-1} b by the generalized eigenvectors of each block's pairs."""
    L = np.linalg.cholesky(M.cpu().numpy())
    Li = np.linalg.inv(L)
    lam, Q = np.linalg.eigh(Li @ P.cpu().numpy() @ np.swapaxes(Li, -1, -2))
    S, lam = _dev(np.swapaxes(Li, -1, -2) @ Q), _dev(lam)
    t = b
    for d in range(3):
        t = _per_block(S[:, d].transpose(1, 2).contiguous(), t, d + 1)
    t = t / (lam[:, 0, :, None, None] + lam[:, 1, None, :, None] + lam[:, 2, None, None, :])
    for d in range(3):
        t = _per_block(S[:, d].contiguous(), t, d + 1)
    return t


def _scaled(p, h):
    """Factor arrays of affine blocks: mass, stiffness, cell operator."""
    hh = h[:, :, None, None]
    M, K, A = (_dev(a) for a in _reference(p))
    return hh * M, K / hh, A / hh


def exact(case, seed):
    kind, groups = case["kind"], _groups(case)
    data = _inputs(case, seed)
    if kind in ("operator", "mgsolve"):
        pairs = [_mesh_1d(case["degree"], m, h, case.get("basis", "lagrange"))
                 for m, h in zip(_cells(case), _mesh_h(case))]
        (Mx, Sx), (My, Sy), (Mz, Sz) = pairs
        if kind == "operator":
            u = _to_grid(case, data["u"].double())
            v = _along(Sx, My, Mz, u)
            v += _along(Mx, Sy, Mz, u)
            v += _along(Mx, My, Sz, u)
            return _blocked(groups, [_from_grid(case, v)])
        V, lam = [], []
        for M, S in pairs:
            Li = np.linalg.inv(np.linalg.cholesky(M))
            w, Q = np.linalg.eigh(Li @ S @ Li.T)
            V.append(Li.T @ Q)
            lam.append(_dev(w))
        t = _along(V[0].T, V[1].T, V[2].T, _to_grid(case, data["b"]))
        t = t / (lam[0][:, None, None] + lam[1][None, :, None] + lam[2][None, None, :])
        return _blocked(groups, [_from_grid(case, _along(V[0], V[1], V[2], t))])
    vs, xs, at = [], [], 0
    for i, (p, nb) in enumerate(groups):
        n = p + 1
        if kind == "factors":
            M, A = data["M"][i], data["P"][i]
            K = A
        else:
            M, K, A = _scaled(p, data["h"][i])
        take = slice(at, at + nb * n ** 3)
        at += nb * n ** 3
        if data["u"] is not None:
            vs.append(_kron_sum(M, K, data["u"][take].double().reshape(nb, n, n, n)))
        xs.append(_kron_solve(M, A, data["b"][take].double().reshape(nb, n, n, n)))
    x = _blocked(groups, xs)
    return x if kind == "solve" else [_blocked(groups, vs), x]
