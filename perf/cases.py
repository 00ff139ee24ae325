"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values.  ``prepare`` makes what a user's program has
in hand before the call (the analysed and bound plan, the values on the GPU),
``run`` makes one pass through the public entry points, ``work`` counts the
bytes and operations the pass cannot do without and ``exact`` gives the
results as dense 64-bit linear algebra has them.

Every case has a ``path``:

* ``solve``: factor + selected inversion of one real matrix (``Plan.factor``,
  ``Plan.invert``), a step of a Newton, self-consistency or sampling loop;
* ``grad``: the differentiable call (``selinv(vals, plan)``) and its backward;
* ``batch``: many independent grids in one plan (``Plan.run``);
* ``poles``: the complex matrices H - z_k S of a pole expansion on one pattern
  (``Plan.factor_complex``, ``Plan.invert_complex``).

and a ``matrix``: ``grid`` (finite-difference Laplacians in two and three
dimensions), ``molecular`` (localized-basis block matrices), ``indefinite``
(saddle-point blocks, 2x2 pivots) or, for poles, a Hamiltonian and an overlap
on the molecular pattern.  The pattern is the case's own: a grid's box, the
sizes of a batch and the atom positions its ``structure`` draws, as a user
keeps one plan over many steps.  The seed draws the values.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1404_0447_amd import selinv as S
from paper_1404_0447_amd import workloads as W

# Diagonal shift of the molecular matrices, which makes them positive definite
# for every seed without an eigenvalue computation.  An unknown couples to at
# most 27 atoms with `dofs` entries of N(0, 1) each: the spectrum of the
# unshifted matrix lies within about 2 sqrt(27 dofs).
MOLECULAR_SHIFT = 2.2


def listed():
    return [
        # the smallest grid of the configurations: a call that is all launches
        # and latency
        dict(name="grid2d_32", path="solve", matrix="grid", dims="32x32", cap=128),
        # a 2D operator (landscape or circuit graph) of ordinary size, sides
        # odd and unequal
        dict(name="grid2d_301x257", path="solve", matrix="grid", dims="301x257", cap=128),
        # a 3D diffusion operator of ordinary size: many levels, most of them
        # with a few hundred tiles
        dict(name="grid3d_40", path="solve", matrix="grid", dims="40x40x40", cap=128),
        # the largest grid of the configurations: throughput of the products
        dict(name="grid3d_64", path="solve", matrix="grid", dims="64x64x64", cap=256),
        # localized-basis electronic structure: dense 8 x 8 blocks, wide
        # supernodes
        dict(name="molecular_16", structure=4, path="solve", matrix="molecular", side=16, dofs=8, cap=128),
        # symmetric indefinite matrix: Bunch-Kaufman pivots in the diagonal
        # blocks
        dict(name="indefinite_12", structure=8, path="solve", matrix="indefinite", side=12, dofs=8, cap=128),
        # fitting a 3D operator's coefficients: forward and backward, box
        # sides odd and unequal
        dict(name="grad_grid3d_31x29x30", path="grad", matrix="grid", dims="31x29x30", cap=128,
             deterministic=False, checkpoint=1),
        # gradients of a molecular matrix, reproducible bit for bit and with
        # the inverse panels checkpointed to save memory between the passes
        dict(name="grad_molecular_9_det", structure=4, path="grad", matrix="molecular", side=9, dofs=8, cap=128,
             deterministic=True, checkpoint=4),
        # many small independent problems of uneven size, replayed as a graph
        dict(name="batch_2d_256", structure=3, path="batch", matrix="grid", count=256, side_lo=32, side_hi=96,
             graph=True),
        # a small batch launched directly
        dict(name="batch_2d_20", structure=3, path="batch", matrix="grid", count=20, side_lo=17, side_hi=61,
             graph=False),
        # a pole expansion: all poles of one pattern in one batch
        dict(name="poles_32", structure=6, path="poles", matrix="pencil", side=10, dofs=8, count=32),
        # one pole alone (a single energy point)
        dict(name="poles_1", structure=6, path="poles", matrix="pencil", side=10, dofs=8, count=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["grid2d", "grid3d", "grid3d", "molecular", "indefinite", "grad_grid", "grad_molecular", "batch",
                       "poles"])
    if kind == "grid2d":
        return dict(path="solve", matrix="grid", dims=f"{_log_int(rng, 24, 400)}x{_log_int(rng, 24, 400)}", cap=128)
    if kind == "grid3d":
        x = _log_int(rng, 8, 56)
        y, z = (max(5, min(56, int(x * rng.uniform(0.6, 1.5)))) for _ in range(2))
        return dict(path="solve", matrix="grid", dims=f"{x}x{y}x{z}", cap=rng.choice([128, 256]))
    if kind in ("molecular", "indefinite"):
        return dict(path="solve", matrix=kind, structure=rng.randrange(1, 1000),
                    side=_log_int(rng, 4, 16 if kind == "molecular" else 12), dofs=rng.choice([4, 6, 8]), cap=128)
    if kind == "grad_grid":
        x = _log_int(rng, 8, 32)
        y, z = (max(5, min(32, int(x * rng.uniform(0.6, 1.4)))) for _ in range(2))
        return dict(path="grad", matrix="grid", dims=f"{x}x{y}x{z}", cap=128, deterministic=rng.random() < 0.25,
                    checkpoint=rng.choice([1, 1, 2, 4]))
    if kind == "grad_molecular":
        return dict(path="grad", matrix="molecular", structure=rng.randrange(1, 1000),
                    side=_log_int(rng, 4, 11), dofs=rng.choice([4, 6, 8]), cap=128,
                    deterministic=rng.random() < 0.25, checkpoint=rng.choice([1, 1, 2, 4]))
    if kind == "batch":
        lo = _log_int(rng, 10, 48)
        return dict(path="batch", matrix="grid", structure=rng.randrange(1, 1000),
                    count=_log_int(rng, 4, 256), side_lo=lo, side_hi=lo + rng.randrange(1, 49),
                    graph=rng.random() < 0.5)
    return dict(path="poles", matrix="pencil", structure=rng.randrange(1, 1000),
                side=_log_int(rng, 4, 10), dofs=rng.choice([4, 6, 8]), count=_log_int(rng, 1, 32))


def _with_values(m, vals):
    return W.Matrix(m.n, m.colptr, m.rowind, vals, ndim=m.ndim, dims=m.dims, dofs=m.dofs)


def _matrix(case, seed):
    """The matrix of a single-matrix case."""
    if case["matrix"] == "grid":
        dims = tuple(int(x) for x in case["dims"].split("x"))
        flat = len(dims) == 2
        return W.laplacian(dims, coeff="uniform" if flat else "loguniform", lo=0.5 if flat else 0.1,
                           hi=2.0 if flat else 10.0, shift=0.01, seed=seed)
    side, dofs, structure = case["side"], case["dofs"], case["structure"]
    if case["matrix"] == "molecular":
        m = W.molecular(side=side, dofs=dofs, seed=structure, shift=0.0)
        v = W.SplitMix64(seed, 1).normal(m.nnz)
        v[m.colptr[:-1]] += MOLECULAR_SHIFT * math.sqrt(27 * dofs)
        return _with_values(m, v)
    # saddle-point self blocks, weak couplings between the atoms
    m = W.indefinite_molecular(side=side, dofs=dofs, seed=structure)
    cols = np.repeat(np.arange(m.n), np.diff(m.colptr))
    between = m.rowind // dofs != cols // dofs
    return _with_values(m, np.where(between, 0.08 * W.SplitMix64(seed, 1).normal(m.nnz), m.vals))


def _batch(case, seed):
    """Grids of the structure's uneven sizes, coefficients and shifts by seed."""
    sizes = W.batch_2d(count=case["count"], side_lo=case["side_lo"], side_hi=case["side_hi"], seed=case["structure"])
    shifts = W.SplitMix64(seed, 0).uniform(len(sizes))
    return [W.laplacian(m.dims[:2], coeff="uniform", lo=0.5, hi=2.0, shift=0.01 + float(x), seed=1000 * seed + i)
            for i, (m, x) in enumerate(zip(sizes, shifts))]


def _pencil(case, seed):
    """H, the values of S on the same pattern, and the poles on a half circle
    around the spectrum."""
    H = W.molecular(side=case["side"], dofs=case["dofs"], seed=case["structure"], shift=0.0)
    H = _with_values(H, W.SplitMix64(seed, 1).normal(H.nnz))
    s = 0.02 * W.SplitMix64(seed, 2).normal(H.nnz)
    s[H.colptr[:-1]] += 1.0
    return H, s, W.poles(case["count"], 0.0, 3.0 * math.sqrt(27 * case["dofs"]))


def _plan(case, what):
    """The analysed plan (host only)."""
    if case["path"] == "batch":
        return S.Plan.batch(what)
    if case["path"] == "poles":
        return S.Plan.poles(what, case["count"])
    kw = dict(max_super=case["cap"])
    if case["path"] == "grad":
        kw.update(deterministic=case["deterministic"], checkpoint_every=case["checkpoint"])
    if case["matrix"] == "indefinite":
        kw.update(pivoting=True)
    return S.Plan.from_matrix(what, **kw)


def _inputs(case, seed):
    """(what the plan is made from, the values on the host)."""
    if case["path"] == "batch":
        ms = _batch(case, seed)
        return ms, np.concatenate([m.vals for m in ms])
    if case["path"] == "poles":
        H, s, z = _pencil(case, seed)
        return H, np.concatenate([H.vals - zk * s for zk in z])
    m = _matrix(case, seed)
    return m, m.vals


def _weights(seed, nnz):
    """The gradient of the user's function by the selected entries."""
    return W.SplitMix64(seed, 3).normal(nnz)


def prepare(case, seed):
    what, vals = _inputs(case, seed)
    plan = _plan(case, what).bind(device="cuda")
    nnzl = int(plan.info["nnzL"])
    vals = torch.as_tensor(vals, device="cuda")
    state = dict(path=case["path"], plan=plan, vals=vals)
    if case["path"] == "grad":
        state["vals"] = vals.requires_grad_(True)
        state["weights"] = torch.as_tensor(_weights(seed, nnzl), device="cuda")
    else:
        state["out"] = torch.empty(nnzl, dtype=vals.dtype, device="cuda")
        state["graph"] = bool(case.get("graph", False))
    return state


def run(state):
    plan, vals = state["plan"], state["vals"]
    if state["path"] == "grad":
        sel = S.selinv(vals, plan)
        (g,) = torch.autograd.grad(sel, vals, state["weights"])
        return dict(selected=sel.detach(), gradient=g)
    if state["path"] == "batch":
        return dict(selected=plan.run(vals, out=state["out"], graph=state["graph"]))
    if state["path"] == "poles":
        plan.factor_complex(vals)
        return dict(selected=plan.invert_complex(state["out"]))
    plan.factor(vals)
    return dict(selected=plan.invert(state["out"]))


@functools.lru_cache(maxsize=None)
def _counts(items):
    case = dict(items)
    what, vals = _inputs(case, 1)
    if case["path"] == "poles":
        case["count"], poles = 1, case["count"]
    else:
        poles = 1
    info = _plan(case, what).info
    return len(vals), poles * int(info["nnzL"]), poles * float(info["flops_factor"] + info["flops_selinv"])


def work(case):
    """Values in, selected entries out, and the multiply-adds of the recurrence
    on the fundamental supernodes (no padding, no explicit zeros).  A complex
    multiply-add is four real ones.  The backward reads the weights, writes a
    gradient, and has two products for each of the forward's."""
    nnza, nnzl, flops = _counts(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    if case["path"] == "poles":
        return dict(bytes=16 * (nnza + nnzl), flops=4.0 * flops)
    if case["path"] == "grad":
        return dict(bytes=8 * (2 * nnza + 2 * nnzl), flops=3.0 * flops)
    return dict(bytes=8 * (nnza + nnzl), flops=flops)


def _inverse(a):
    """Dense inverse by 2 x 2 blocks (Schur complements), leaves by a library
    inverse: nearly all of it matrix products."""
    n = a.shape[0]
    if n <= 1024:
        return torch.linalg.inv(a)
    h = n // 2
    ai = _inverse(a[:h, :h])
    w = ai @ a[:h, h:].contiguous()
    si = _inverse(a[h:, h:] - a[h:, :h].contiguous() @ w)
    wsi = w @ si
    out = torch.empty_like(a)
    out[h:, h:] = si
    out[:h, h:] = -wsi
    out[h:, :h] = -wsi.t()  # A is symmetric (not Hermitian where complex)
    out[:h, :h] = ai + wsi @ w.t().contiguous()
    return out


def _dense(m, vals, device):
    cols = np.repeat(np.arange(m.n), np.diff(m.colptr))
    rows = torch.as_tensor(m.rowind.astype(np.int64), device=device)
    cols = torch.as_tensor(cols, device=device)
    v = torch.as_tensor(vals, device=device)
    a = torch.zeros(m.n, m.n, dtype=v.dtype, device=device)
    a[rows, cols] = v
    a[cols, rows] = v
    return a, rows, cols


def _selected_positions(m, pattern, device):
    """Original (row, column) of every entry of the selected pattern."""
    cp, ri, perm = pattern
    cols = np.repeat(np.arange(m.n), np.diff(cp))
    p = perm.astype(np.int64)
    return torch.as_tensor(p[ri], device=device), torch.as_tensor(p[cols], device=device)


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    limit = 34000 if device == "cuda" else 3000
    what, vals = _inputs(case, seed)
    if case["path"] == "batch":
        if sum(m.n ** 3 for m in what) > limit ** 3:
            return None
        parts = []
        for m in what:
            a, _, _ = _dense(m, m.vals, device)
            i, j = _selected_positions(m, S.Plan.from_matrix(m).pattern(), device)
            parts.append(_inverse(a)[i, j])
        return dict(selected=torch.cat(parts))
    if case["path"] == "poles":
        if 2 * case["count"] * what.n ** 3 > limit ** 3:
            return None
        one = _plan({**case, "count": 1}, what).pattern()
        i, j = _selected_positions(what, one, device)
        parts = []
        for v in vals.reshape(case["count"], -1):
            a, _, _ = _dense(what, v, device)
            parts.append(_inverse(a)[i, j])
        return dict(selected=torch.cat(parts))
    if what.n > limit:
        return None
    a, rows, cols = _dense(what, vals, device)
    # a saddle-point matrix needs pivots across the blocks
    x = torch.linalg.inv(a) if case["matrix"] == "indefinite" else _inverse(a)
    i, j = _selected_positions(what, _plan(case, what).pattern(), device)
    out = dict(selected=x[i, j])
    if case["path"] == "grad":
        # f = sum of w * Ainv over the selected entries; an off-diagonal entry
        # of A drives both of its places, a diagonal one its own
        w = torch.as_tensor(_weights(seed, len(i)), device=device)
        g = torch.zeros_like(a)
        g.index_put_((i, j), w, accumulate=True)
        g.index_put_((j, i), w, accumulate=True)
        d = -(x @ g @ x)[rows, cols]
        out["gradient"] = torch.where(rows == cols, 0.5 * d, d)
    return out
