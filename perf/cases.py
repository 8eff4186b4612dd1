"""Workloads whose speed is tracked, through the public Python entry points.

Each case is one pass a program makes again and again on a pattern it has
analysed once:

    op "step"     refactorize with the state's values, then solve (time steps,
                  Newton steps: same pattern, new values)
    op "solve"    solve with a resident factor
    op "refined"  low-precision refactorize, then a solve refined to FP64
    op "resolve"  refined solve with a resident low-precision factor (the
                  re-solve requests of the serving workload)
    op "batch"    factorize a batch of independent systems and solve it (FP64)
                  or solve it refined to FP64 (FP32)

The operators are the repository's grid families: "grid2d" (5-point),
"grid3d" (7-point), both with conductances 10^U[-2, 2), and "elast" (27-point,
3 degrees of freedom per point, random symmetric edge blocks).  Every case
takes the schedule that the library chooses by itself (no tuned cut-offs), as
a program does on a size that nobody has tuned.
"""
import functools
import math

import numpy as np
import torch

from paper_2202_09288_amd import spchol
from paper_2202_09288_amd import workloads as W

_SHIFT = 1e-2   # diagonal shift of the scalar operators (the batch workload's)
_KAPPA = 1e6    # condition number aimed at by the elasticity operator's shift
_TOL = 1e-14    # backward error of refined solves: that of a plain FP64 solve, with room
_STENCIL = {"grid2d": "5pt", "grid3d": "7pt", "elast": "27pt"}


def _one(name, op, kind, nx, ny, nz, nrhs, precision, graph=False):
    return {"name": name, "op": op, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "nrhs": nrhs,
            "precision": precision, "graph": graph}


def _batch(name, count, mix, nrhs, precision):
    return {"name": name, "op": "batch", "count": count, "mix": mix, "nrhs": nrhs, "precision": precision}


def listed():
    return [
        # one right-hand side on the smallest 2D member of the batch mix: latency of a re-solve
        _one("solve_2d_32", "solve", "grid2d", 32, 32, 1, 1, "fp64"),
        # the smallest benchmark configuration, replayed from a graph as its benchmark does
        _one("step_2d_64", "step", "grid2d", 64, 64, 1, 1, "fp64", True),
        # the largest 2D member of the batch mix, eager, a few right-hand sides
        _one("step_2d_200", "step", "grid2d", 200, 200, 1, 8, "fp64"),
        # an ordinary small 3D problem on a ragged grid, eager
        _one("step_3d_21", "step", "grid3d", 21, 20, 19, 3, "fp64"),
        # the largest 3D member of the batch mix alone, mixed precision, a full chunk of right-hand sides
        _one("refined_3d_34", "refined", "grid3d", 34, 34, 34, 16, "fp32"),
        # the serving workload's re-solve of its largest system
        _one("resolve_3d_50", "resolve", "grid3d", 50, 50, 50, 8, "fp32"),
        # the 60^3 benchmark configuration: factor plus solve, and its solve alone
        _one("step_3d_60", "step", "grid3d", 60, 60, 60, 1, "fp64", True),
        _one("solve_3d_60", "solve", "grid3d", 60, 60, 60, 1, "fp64"),
        # structural solves: many load cases on a resident factor
        _one("solve_elast_30", "solve", "elast", 30, 29, 27, 16, "fp64"),
        # BF16 Schur updates recovered to FP64 by refinement
        _one("refined_elast_20", "refined", "elast", 20, 20, 20, 4, "bf16upd"),
        # the headline benchmark configuration
        _one("step_elast_48", "step", "elast", 48, 48, 48, 4, "fp64", True),
        # uneven batch of independent systems, refined
        _batch("batch_32", 32, 0, 16, "fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: ragged sides, 1 to 17 right-hand sides."""
    op = rng.choice(["step", "step", "step", "solve", "solve", "refined", "resolve", "batch"])
    nrhs = rng.choice([1, 1, 2, 3, 4, 5, 8, 11, 16, 17])
    if op == "batch":
        c = _batch("", _log(rng, 4, 32), rng.randrange(1, 1 << 20), nrhs, rng.choice(["fp64", "fp32"]))
    else:
        kind = rng.choice(["grid2d", "grid3d", "grid3d", "elast"])
        lo, hi = {"grid2d": (32, 200), "grid3d": (10, 60), "elast": (6, 40)}[kind]
        side = _log(rng, lo, hi)
        nx, ny, nz = (max(lo - 2, side - rng.randrange(0, 4)) for _ in range(3))
        precision = "fp64" if op in ("step", "solve") else rng.choice(["fp32", "fp32", "bf16upd"])
        c = _one("", op, kind, nx, ny, nz if kind != "grid2d" else 1, nrhs, precision, rng.random() < 0.5)
    del c["name"]
    return c


# ----------------------------------------------------------------------------
# patterns (one analysis per pattern and process, as a program keeps it) and
# values from a seed
# ----------------------------------------------------------------------------

class _Pattern:
    """Lower-CSC pattern of a grid operator, where each edge's values go in
    it, and its analysis."""

    def __init__(self, kind, dims):
        self.kind, self.dof = kind, 3 if kind == "elast" else 1
        d, npts = self.dof, int(np.prod(dims))
        self.npts, self.n = npts, d * npts
        hi, lo = (torch.from_numpy(a) for a in W.grid_edges(dims, _STENCIL[kind]))
        # the edges of one stencil offset touch each point at most once per end
        node, axes = np.arange(npts), []
        for s in dims:
            axes.append(node % s)
            node = node // s
        axes = [torch.from_numpy(a) for a in axes]
        code = sum((axes[a][hi] - axes[a][lo] + 1) * 3 ** a for a in range(len(dims)))
        self.groups = [(code == c).nonzero().flatten() for c in code.unique().tolist()]
        b = torch.arange(d)
        bi, bj = (t.reshape(-1) for t in torch.meshgrid(b, b, indexing="ij"))
        low = bi >= bj
        pts = torch.arange(npts)
        rows = torch.cat([(d * pts[:, None] + bi[low]).reshape(-1), (d * hi[:, None] + bi).reshape(-1)])
        cols = torch.cat([(d * pts[:, None] + bj[low]).reshape(-1), (d * lo[:, None] + bj).reshape(-1)])
        key = (cols * self.n + rows).cuda().sort()
        place = torch.empty_like(key.indices)
        place[key.indices] = torch.arange(place.numel(), device="cuda")
        colptr = np.concatenate([[0], np.bincount((key.values // self.n).cpu().numpy(), minlength=self.n).cumsum()])
        rowidx = (key.values % self.n).to(torch.int32).cpu().numpy()
        self.colptr, self.rowidx = colptr, rowidx
        self.hi, self.lo, self.low, self.place = hi.cuda(), lo.cuda(), low.cuda(), place
        self.groups = [g.cuda() for g in self.groups]
        self.sym = spchol.analyze(colptr, rowidx, W.nd_perm(dims, dof=d))

    def values(self, gen):
        ne, d = self.hi.numel(), self.dof

        def rand(*shape):
            return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=gen)

        lam = 10.0 ** (4.0 * rand(ne, d) - 2.0)
        if d == 1:
            K = lam
        else:  # Q diag(lam) Q^T with Q the rotation of a random unit quaternion
            w, x, y, z = torch.nn.functional.normalize(2.0 * rand(4, ne) - 1.0, dim=0)
            Q = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                             2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                             2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(ne, 3, 3)
            K = sum(lam[:, k, None, None] * Q[:, :, k, None] * Q[:, None, :, k] for k in range(3)).reshape(ne, 9)
        diag = torch.zeros(self.npts, d * d, dtype=torch.float64, device="cuda")
        for g in self.groups:
            diag[self.hi[g]] += K[g]
            diag[self.lo[g]] += K[g]
        eye = torch.eye(d, dtype=torch.float64, device="cuda").reshape(-1)
        shift = _SHIFT if d == 1 else 2.0 * diag.abs().sum(1).max() / _KAPPA
        out = torch.empty(self.place.numel(), dtype=torch.float64, device="cuda")
        out[self.place] = torch.cat([(diag + shift * eye)[:, self.low].reshape(-1), -K.reshape(-1)])
        return out


@functools.lru_cache(maxsize=4)
def _pattern(kind, dims):
    return _Pattern(kind, dims)


@functools.lru_cache(maxsize=1)
def _batch_patterns(count, mix):
    made = {}
    for kind, side in W.batch_specs(count, mix):
        dims = (side, side) if kind == "2d" else (side, side, side)
        if dims not in made:
            made[dims] = _Pattern("grid" + kind, dims)
    return [made[(s, s) if k == "2d" else (s, s, s)] for k, s in W.batch_specs(count, mix)]


def _dims(case):
    return (case["nx"], case["ny"]) if case["kind"] == "grid2d" else (case["nx"], case["ny"], case["nz"])


def _patterns(case):
    return _batch_patterns(case["count"], case["mix"]) if case["op"] == "batch" else [_pattern(case["kind"], _dims(case))]


def _inputs(case, seed):
    """(pattern, values, right-hand sides) of each system of the case."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = []
    for p in _patterns(case):
        v = p.values(gen)
        b = 2.0 * torch.rand(case["nrhs"], p.n, dtype=torch.float64, device="cuda", generator=gen) - 1.0
        out.append((p, v, b))
    return out


def prepare(case, seed):
    systems = _inputs(case, seed)
    s = {"op": case["op"], "precision": case["precision"], "v": [v for _, v, _ in systems],
         "b": [b for _, _, b in systems], "x": [torch.empty_like(b) for _, _, b in systems]}
    if case["op"] == "batch":
        s["batch"] = spchol.Batch([p.sym for p, _, _ in systems], case["precision"])
        s["batch"].factorize(s["v"])
        s["batch"].sync()
    else:
        s["f"] = spchol.factorize(systems[0][0].sym, s["v"][0], case["precision"])
        s["f"].sync()
        if case["graph"]:
            s["f"].set_graph(True)
    return s


def run(s):
    if s["op"] == "batch":
        s["batch"].factorize(s["v"])
        if s["precision"] == "fp64":
            for x, b in zip(s["x"], s["b"]):
                x.copy_(b)
            s["batch"].solve(s["x"])
        else:
            s["batch"].solve_refined(s["b"], s["x"], tol=_TOL, maxit=60)
        return s["x"]
    f, v, b, x = s["f"], s["v"][0], s["b"][0], s["x"][0]
    if s["op"] in ("step", "refined"):
        f.refactorize(v)
    if s["op"] in ("step", "solve"):
        x.copy_(b)
        f.solve(x)
    else:
        f.solve_refined(v, b, x, tol=_TOL, maxit=60)
    return x


def work(case):
    """Factoring reads A's values and writes L; solving reads B, reads L (a
    resident factor), writes X; a refined solve reads A once more."""
    entry = 8 if case["precision"] == "fp64" else 4
    nrhs, nbytes, flops = case["nrhs"], 0.0, 0.0
    for p in _patterns(case):
        i = p.sym.info
        nbytes += 16.0 * i["n"] * nrhs + entry * i["nnz_l"]
        flops += 4.0 * i["nnz_l"] * nrhs
        if case["op"] in ("step", "refined", "batch"):
            nbytes += 8.0 * i["nnz_a"]
            flops += i["flops"]
        if case["op"] == "resolve":
            nbytes += 8.0 * i["nnz_a"]
        if case["precision"] != "fp64":
            flops += 4.0 * i["nnz_a"] * nrhs
    return {"bytes": nbytes, "flops": flops}


# ----------------------------------------------------------------------------
# the solutions in 64 bits, by plain torch
# ----------------------------------------------------------------------------

def _full(p, v):
    """The full symmetric matrix of lower-CSC values, as sparse CSR."""
    cols = torch.repeat_interleave(torch.arange(p.n, device="cuda"),
                                   torch.from_numpy(np.diff(p.colptr)).cuda())
    rows = torch.from_numpy(p.rowidx).cuda().long()
    off = rows != cols
    idx = torch.stack([torch.cat([rows, cols[off]]), torch.cat([cols, rows[off]])])
    return torch.sparse_coo_tensor(idx, torch.cat([v, v[off]]), (p.n, p.n)).coalesce().to_sparse_csr()


def _cg(A, d, B, steps):
    """X = A^{-1} B by conjugate gradients with the diagonal d, restarted on
    the true residual, and the residual it ends with."""
    X = torch.zeros_like(B)
    best, kept = math.inf, X
    for _ in range(6):
        R = B - A @ X
        now = (R.abs().amax(0) / B.abs().amax(0)).max().item()
        if now < best:
            best, kept = now, X.clone()
        elif now > 0.5 * best:
            break
        Z = R / d
        P, rho = Z.clone(), (R * Z).sum(0)
        goal = 1e-8 * rho
        for k in range(steps):
            Q = A @ P
            a = rho / (P * Q).sum(0)
            X = X + a * P
            R = R - a * Q
            Z = R / d
            new = (R * Z).sum(0)
            if k % 50 == 49 and bool((new <= 1e-6 * goal).all()):
                break
            P = Z + torch.nan_to_num(new / rho) * P
            rho = new
    return kept, best


def exact(case, seed):
    """Dense Cholesky up to n = 12000, conjugate gradients beyond for the
    scalar operators (the elasticity operators would take too many steps)."""
    if case["op"] != "batch" and case["kind"] == "elast" and 3 * math.prod(_dims(case)) > 12000:
        return None
    out = []
    for p, v, b in _inputs(case, seed):
        A, B = _full(p, v), b.T.contiguous()
        if p.n <= 12000:
            x = torch.cholesky_solve(B, torch.linalg.cholesky(A.to_dense()))
        else:
            x, left = _cg(A, v[torch.from_numpy(p.colptr[:-1]).cuda()][:, None], B, 6000)
            if left > 1e-11:
                return None
        out.append(x.T.contiguous())
    return out if case["op"] == "batch" else out[0]
