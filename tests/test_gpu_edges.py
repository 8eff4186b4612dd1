"""GPU kernels at the edges of their tiles, against the CPU oracle: panels and
blocks of 1 to a few columns and rows, one row or column past a tile, every
level launched on its own and every level persistent.

Tolerances: solves are held to the normwise backward error 1e-12 (FP64) and
1e-5 (FP32), factors to 1e-10 (FP64, each supernode on its own), the bars of
the other parity tests.
"""
import numpy as np
import pytest

import oracle
from paper_2202_09288_amd import workloads as W
from tests.wide_levels import BORDER, WIDTHS, uneven_arrow

pytestmark = pytest.mark.gpu

BAR = {"fp64": 1e-12, "fp32": 1e-5}


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2202_09288_amd import spchol
    return spchol


def spd(n, pattern, seed=0):
    """Diagonally dominant matrix with the given strictly lower entries."""
    rng = np.random.default_rng(seed)
    r, c = pattern
    v = -(0.5 + rng.random(r.size))
    d = 1.0 + np.bincount(r, -v, n) + np.bincount(c, -v, n)
    colptr, rowidx, values = W.lower_csc(n, np.concatenate([np.arange(n), r]), np.concatenate([np.arange(n), c]),
                                         np.concatenate([d, v]))
    return colptr, rowidx, values, np.arange(n, dtype=np.int32)


def dense(n):
    return spd(n, np.tril_indices(n, -1))


def wide(w, m):
    """One supernode of w columns and m rows, over a dense trailing block."""
    return spd(m, np.tril_indices(m, -1)) if w == m else spd(
        m, tuple(np.concatenate(a) for a in zip(np.tril_indices(w, -1),
                                                (np.repeat(np.arange(w, m), w), np.tile(np.arange(w), m - w)))))


def tridiag(n):
    return spd(n, (np.arange(1, n), np.arange(n - 1)))


MATRICES = {
    "one": lambda: dense(1), "pair": lambda: dense(2), "triple": lambda: dense(3), "tridiag-5": lambda: tridiag(5),
    "dense-63": lambda: dense(63), "dense-65": lambda: dense(65), "dense-130": lambda: dense(130),
    "wide-17x18": lambda: wide(17, 18), "wide-64x321": lambda: wide(64, 321), "wide-66x323": lambda: wide(66, 323),
}
# every supernode on the blocked paths
BLOCKED = {"tiny_w": -1, "tiny_m": -1, "small_w": -1, "small_m": -1}


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(MATRICES))
def test_solve_sweeps_on_ragged_blocks(lib, name, precision):
    """The block sweeps' wide loads, row and column tiles and right-hand-side
    padding on blocks and tasks that fill them only in part."""
    import torch
    colptr, rowidx, values, perm = MATRICES[name]()
    n = colptr.size - 1
    B = np.random.default_rng(3).uniform(-1, 1, (n, 17))
    dv = torch.from_numpy(values).cuda()
    for persist in (-1, 1 << 30):
        F = lib.factorize(lib.Symbolic(colptr, rowidx, perm, 0.05, dict(BLOCKED, solve_persist_max=persist)), dv,
                          precision)
        F.sync()
        for q in (1, 2, 4, 9, 16, 17):
            X = torch.from_numpy(np.ascontiguousarray(B[:, :q].T)).cuda()
            F.solve(X)
            F.sync()
            eta = oracle.backward_error(n, colptr, rowidx, values, X.cpu().numpy().T, B[:, :q])
            print(f"{name} {precision} persist={persist} nrhs={q}: eta={eta:.2e}", flush=True)
            assert eta <= BAR[precision]


def arrow(w, b, blocks=2):
    """Dense blocks of w columns, each coupled to the same b last columns:
    supernodes of w columns and w + b rows, and one of b columns."""
    n = blocks * w + b
    rows, cols = [], []
    for k in range(blocks):
        r, c = np.tril_indices(w, -1)
        rows += [k * w + r, blocks * w + np.repeat(np.arange(b), w)]
        cols += [k * w + c, k * w + np.tile(np.arange(w), b)]
    return spd(n, (np.concatenate(rows), np.concatenate(cols)), seed=w)


def factor_and_solve(lib, matrix, tuning, precision="fp64", nrhs=3, z=-1.0):
    """Largest relative error of a supernode against the oracle, and the
    solve's backward error."""
    import torch
    colptr, rowidx, values, perm = matrix
    n = colptr.size - 1
    S = oracle.Symbolic(colptr, rowidx, perm, z)
    F = lib.factorize(lib.Symbolic(colptr, rowidx, perm, z, tuning), torch.from_numpy(values).cuda(), precision)
    F.sync()
    per = oracle.supernode_rel_errors(F.export(), S.factor(values), S.lptr, S.lower_mask())
    B = np.random.default_rng(4).uniform(-1, 1, (n, nrhs))
    X = torch.from_numpy(np.ascontiguousarray(B.T)).cuda()
    F.solve(X)
    F.sync()
    return float(per.max()), oracle.backward_error(n, colptr, rowidx, values, X.cpu().numpy().T, B), S


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("persist", [-1, 1])
@pytest.mark.parametrize("w,b", [(1, 127), (1, 1), (9, 40), (15, 113), (16, 112), (17, 111), (17, 1), (20, 33),
                                 (31, 97), (32, 96), (32, 1), (30, 50)])
def test_small_supernode_shapes(lib, w, b, persist, precision):
    """The one-workgroup path at one and two 16-column panels, ragged ones
    among them, and at the fewest and most rows below."""
    err, eta, S = factor_and_solve(lib, arrow(w, b), {"tiny_w": -1, "persist": persist}, precision)
    print(f"w={w} b={b} persist={persist} {precision}: worst supernode {err:.2e}, eta {eta:.2e}", flush=True)
    assert S.nsuper == 3 and err <= (1e-10 if precision == "fp64" else 1e-4) and eta <= BAR[precision]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 33, 48, 49, 63, 64, 65, 80, 127, 129, 193])
def test_diagonal_block_shapes(lib, n, precision):
    """The factorization of a 64-column block at one to four 16-column panels,
    full and ragged, alone and after other blocks of its supernode."""
    err, eta, S = factor_and_solve(lib, dense(n), BLOCKED, precision)
    print(f"n={n} {precision}: worst supernode {err:.2e}, eta {eta:.2e}", flush=True)
    assert err <= (1e-10 if precision == "fp64" else 1e-4) and eta <= BAR[precision]


@pytest.mark.parametrize("precision,scale", [("fp64", 2.0 ** 1010), ("fp64", 2.0 ** -1000), ("fp32", 2.0 ** 119),
                                             ("fp32", 2.0 ** -110)])
@pytest.mark.parametrize("tuning", [{}, BLOCKED], ids=["small", "blocked"])
def test_values_near_the_ends_of_the_range(lib, tuning, precision, scale):
    """Pivots near the largest and smallest normal numbers of the precision:
    the factor scales with the square root of the matrix."""
    colptr, rowidx, values, perm = arrow(20, 30)
    err, _, _ = factor_and_solve(lib, (colptr, rowidx, values * scale, perm), tuning, precision)
    print(f"{precision} scale {scale:.1e} {tuning}: worst supernode {err:.2e}", flush=True)
    assert err <= (1e-10 if precision == "fp64" else 1e-4)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("group", [1, -1])
@pytest.mark.parametrize("w,b", [(1, 1), (1, 15), (2, 14), (4, 12), (4, 13), (3, 29), (4, 28), (1, 63), (5, 16),
                                 (8, 17), (8, 33), (8, 56), (7, 49), (8, 0)])
def test_tiny_supernode_shapes(lib, w, b, group, precision):
    """Tiny supernodes at the edges of the 16-lane, 32-lane and one-wave forms
    and of their 16-row tiles; the border's supernode is tiny, small or
    blocked beside them."""
    matrix = arrow(w, b, blocks=5) if b else arrow(w, 1, blocks=9)
    err, eta, _ = factor_and_solve(lib, matrix, {"group": group}, precision)
    print(f"w={w} b={b} group={group} {precision}: worst supernode {err:.2e}, eta {eta:.2e}", flush=True)
    assert err <= (1e-10 if precision == "fp64" else 1e-4) and eta <= BAR[precision]


def test_default_groups_of_blocks(lib):
    """Levels with enough trailing tiles take groups of four column blocks by
    default, on every supernode of the level, ragged last blocks included:
    the factor is the oracle's and that of one block a group."""
    matrix = arrow(700, 8, blocks=64)
    for tuning in ({}, {"delay": 1}, {"lookahead": -1}, {"handover": -1}):
        err, eta, S = factor_and_solve(lib, matrix, tuning, nrhs=1)
        print(f"{tuning}: worst supernode {err:.2e}, eta {eta:.2e}", flush=True)
        assert S.nsuper == 65 and err <= 1e-10 and eta <= BAR["fp64"]


def tridiag_errors(n, values, X, B):
    """Backward error of each column for a tridiagonal matrix (lower CSC)."""
    d, e = values[0::2], values[1::2]  # the columns hold (diagonal, below)
    AX = d[:, None] * X
    AX[1:] += e[:, None] * X[:-1]
    AX[:-1] += e[:, None] * X[1:]
    rows = np.abs(d)
    rows[1:] += np.abs(e)
    rows[:-1] += np.abs(e)
    return np.abs(B - AX).max(0) / (rows.max() * np.abs(X).max(0) + np.abs(B).max(0))


@pytest.mark.parametrize("maxit", [0, 4])
@pytest.mark.parametrize("sizes", [(1,), (255,), (1023,), (1024,), (1025,), (2050,), (1, 1023), (700, 324, 1, 1024, 3),
                                   (40, 1, 2, 61, 64, 1300), (3000, 1, 5000)], ids=str)
@pytest.mark.parametrize("nrhs", [1, 2, 3, 5, 8, 9, 17])
def test_refinement_reductions(lib, sizes, nrhs, maxit):
    """Refinement of one system and of batches whose systems end inside and
    at the chunks of the reductions, over the column counts of the SpMV: the
    reported backward error is the one taken on the host.  Both residuals are
    of three products in FP64, so the two differ by at most a few units of
    roundoff of |A||x| + |b|: 2e-15.  With tol = 0 the steps (refinement, then
    conjugate gradients) only end at maxit."""
    import torch
    systems = [tridiag(n) if n > 1 else dense(1) for n in sizes]
    rng = np.random.default_rng(nrhs)
    Bh = [rng.standard_normal((nrhs, n)) * 10.0 ** rng.integers(-3, 4, (nrhs, 1)) for n in sizes]
    syms = [lib.Symbolic(c, r, p, 0.0) for c, r, _, p in systems]
    vals = [torch.from_numpy(v).cuda() for _, _, v, _ in systems]
    Bs = [torch.from_numpy(b).cuda() for b in Bh]
    Xs = [torch.zeros_like(b) for b in Bs]
    if len(sizes) == 1:
        F = lib.factorize(syms[0], vals[0], "fp32")
        out = [F.solve_refined(vals[0], Bs[0], Xs[0], tol=0.0, maxit=maxit)]
    else:
        batch = lib.Batch(syms, "fp32")
        batch.factorize(vals)
        out = batch.solve_refined(Bs, Xs, tol=0.0, maxit=maxit)["systems"]
    for n, (_, _, v, _), b, x, r in zip(sizes, systems, Bh, Xs, out):
        eta = tridiag_errors(n, v, x.cpu().numpy().T, b.T).max()
        print(f"n={n} nrhs={nrhs} maxit={maxit}: reported {r['berr']:.3e}, host {eta:.3e}", flush=True)
        assert abs(r["berr"] - eta) <= 2e-15
        assert eta <= (1e-5 if maxit == 0 else 1e-14)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tiny", [1, 3, 6, 16380, 16388])
def test_solve_levels_of_tiny_and_wide_supernodes(lib, tiny, precision):
    """A solve level that holds both kinds: its tiny supernodes share the
    block tasks' launch up to 4096 workgroups of four and have one of their
    own beyond, with ragged last workgroups in both."""
    import torch
    w, b, wide_w, wide_blocks = 3, 20, 40, 3
    n = tiny * w + wide_blocks * wide_w + b
    rows, cols, c0 = [], [], 0
    for width in [w] * tiny + [wide_w] * wide_blocks + [b]:
        r, c = np.tril_indices(width, -1)
        rows.append(c0 + r)
        cols.append(c0 + c)
        if c0 + width < n:  # coupled to the last b columns
            rows.append(n - b + np.repeat(np.arange(b), width))
            cols.append(c0 + np.tile(np.arange(width), b))
        c0 += width
    colptr, rowidx, values, perm = spd(n, (np.concatenate(rows), np.concatenate(cols)))
    sym = lib.Symbolic(colptr, rowidx, perm, -1.0, {"solve_persist_max": -1})
    F = lib.factorize(sym, torch.from_numpy(values).cuda(), precision)
    F.sync()
    B = np.random.default_rng(5).uniform(-1, 1, (n, 16))
    for q in (1, 3, 16):
        X = torch.from_numpy(np.ascontiguousarray(B[:, :q].T)).cuda()
        F.solve(X)
        F.sync()
        eta = oracle.backward_error(n, colptr, rowidx, values, X.cpu().numpy().T, B[:, :q])
        print(f"tiny={tiny} {precision} nrhs={q}: eta={eta:.2e}", flush=True)
        assert eta <= BAR[precision]


def exponents(kind, n, precision):
    """Powers of two for the rows and columns: `ends` mixes diagonals near both
    ends of the precision's range in every tile, `one` puts a single large one
    among small ones, `random` spreads them, `subnormal` puts all of them below
    the normal numbers."""
    top = 505 if precision == "fp64" else 59
    i = np.arange(n)
    return {"ends": np.where(i % 2, top - 4, 4 - top), "one": np.where(i == 3, top, -3 * top // 4),
            "random": np.random.default_rng(n).integers(5 - top, top - 5, n),
            "subnormal": np.full(n, -515 if precision == "fp64" else -66)}[kind]


def scaled_factor_error(lib, n, kind, precision, tuning):
    """Largest error of a row of the factor of S B S, relative to the row, S
    powers of two and B well conditioned (of a few bits, so that S B S is
    exact down into the subnormal numbers): the factor is S times that of B."""
    import torch
    B = np.tril(np.random.default_rng(n).integers(-8, 9, (n, n)) / 16.0, -1)
    B = B + B.T
    B[np.diag_indices(n)] = np.ceil(np.abs(B).sum(1)) + 1
    s = np.exp2(exponents(kind, n, precision))
    r, c = np.tril_indices(n)
    colptr, rowidx, values = W.lower_csc(n, r, c, B[r, c] * s[r] * s[c])
    sym = lib.Symbolic(colptr, rowidx, np.arange(n, dtype=np.int32), 0.05, tuning)
    F = lib.factorize(sym, torch.from_numpy(values).cuda(), precision)
    F.sync()
    ref = np.linalg.cholesky(B)
    L = np.tril(F.export().reshape(n, n).T) / s[:, None]
    b = np.random.default_rng(7).uniform(-1, 1, n)
    X = torch.from_numpy((b * s)[None, :].copy()).cuda()
    F.solve(X)
    F.sync()
    x = X.cpu().numpy()[0] * s
    return float((np.linalg.norm(L - ref, axis=1) / np.linalg.norm(ref, axis=1)).max()), \
        float(np.abs(B @ x - b).max() / (np.abs(B).sum(1).max() * np.abs(x).max() + np.abs(b).max()))


@pytest.mark.parametrize("precision,kind", [("fp64", "ends"), ("fp64", "one"), ("fp64", "random"),
                                            ("fp64", "subnormal"), ("fp32", "ends"), ("fp32", "one"),
                                            ("fp32", "random"), ("bf16upd", "ends"), ("bf16upd", "one")])
@pytest.mark.parametrize("n", [8, 24, 40, 193])
def test_blocks_of_pivots_of_different_magnitude(lib, n, kind, precision):
    """Diagonals of one 16-column tile far apart, and near the ends of the
    range: the 64-column blocks' factorization loses nothing by it.  (With BF16
    updates the blocks after the first are only good to the rounding of their
    operands, 2^-8.)"""
    err, eta = scaled_factor_error(lib, n, kind, precision, BLOCKED)
    print(f"n={n} {kind} {precision}: worst row {err:.2e}, eta {eta:.2e}", flush=True)
    rough = precision == "bf16upd" and n > 64
    assert err <= (1e-2 if rough else 1e-10 if precision == "fp64" else 1e-4)
    assert eta <= (1e-2 if rough else BAR["fp64" if precision == "fp64" else "fp32"])


@pytest.mark.parametrize("kind", ["ends", "one", "random", "subnormal"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,persist", [(9, -1), (17, 1), (32, -1)])
def test_small_supernodes_of_pivots_of_different_magnitude(lib, n, persist, precision, kind):
    """The same for the one-workgroup path."""
    err, eta = scaled_factor_error(lib, n, kind, precision, {"tiny_w": -1, "tiny_m": -1, "persist": persist})
    print(f"n={n} {kind} {precision} persist={persist}: worst row {err:.2e}, eta {eta:.2e}", flush=True)
    assert err <= (1e-10 if precision == "fp64" else 1e-4) and eta <= BAR[precision]


@pytest.fixture(scope="module")
def uneven():
    """The wide level of tests/wide_levels.py as one system and as two."""
    return uneven_arrow(sum(WIDTHS, []), BORDER), [uneven_arrow(w, BORDER, i) for i, w in enumerate(WIDTHS)]


def csc_backward_error(matrix, X, B):
    """Normwise backward error (largest column) of a lower CSC system."""
    import scipy.sparse as sp
    colptr, rowidx, values, _ = matrix
    n = colptr.size - 1
    A = sp.csc_matrix((values, rowidx, colptr), shape=(n, n))
    A = A + sp.tril(A, -1).T
    r = np.abs(B - A @ X).max(0)
    return float((r / (abs(A).sum(1).max() * np.abs(X).max(0) + np.abs(B).max(0))).max())


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16upd"])
def test_default_groups_follow_each_other(lib, uneven, precision):
    """Two default groups of four blocks in a row with supernodes that end
    raggedly inside them: the factor is that of one block a group, to the
    rounding of the updates (BF16 operands: 2^-8), with the update beyond the
    next group spread over its steps or not, on 128x128 tiles, and under every
    hand-over rule."""
    import torch
    colptr, rowidx, values, perm = uneven[0]
    n = colptr.size - 1
    dv = torch.from_numpy(values).cuda()
    B = np.random.default_rng(9).uniform(-1, 1, (n, 3))
    bar = {"fp64": (1e-10, 1e-12), "fp32": (1e-4, 1e-5), "bf16upd": (1e-2, 1e-2)}[precision]
    ref = None
    for tuning in ({"delay": 1}, {}, {"lookahead": -1}, {"handover": 1}, {"handover": -1}, {"bulk128": 1}):
        sym = lib.Symbolic(colptr, rowidx, perm, -1.0, tuning)
        F = lib.factorize(sym, dv, precision)
        F.sync()
        L = F.export()
        if ref is None:
            ref, lptr = L, oracle.Symbolic(colptr, rowidx, perm, -1.0).lptr
        err = float(oracle.supernode_rel_errors(L, ref, lptr).max())
        X = torch.from_numpy(np.ascontiguousarray(B.T)).cuda()
        F.solve(X)
        F.sync()
        eta = csc_backward_error(uneven[0], X.cpu().numpy().T, B)
        print(f"{precision} {tuning}: worst supernode {err:.2e}, eta {eta:.2e}", flush=True)
        assert err <= bar[0] and eta <= bar[1]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16upd"])
def test_default_groups_of_a_batch(lib, uneven, precision):
    """Two systems whose merged level reaches the groups' limit, which neither
    reaches alone, also when factored again."""
    import torch
    systems = uneven[1]
    vals = [torch.from_numpy(v).cuda() for _, _, v, _ in systems]
    Bs = [np.random.default_rng(i).uniform(-1, 1, (2, c.size - 1)) for i, (c, _, _, _) in enumerate(systems)]
    batch = lib.Batch([lib.Symbolic(c, r, p, -1.0) for c, r, _, p in systems], precision)
    for _ in range(2):
        batch.factorize(vals)
        Xs = [torch.from_numpy(b).cuda() for b in Bs]
        batch.solve(Xs)
        batch.sync()
        for matrix, x, b in zip(systems, Xs, Bs):
            eta = csc_backward_error(matrix, x.cpu().numpy().T, b.T)
            print(f"{precision} n={b.shape[1]}: eta {eta:.2e}", flush=True)
            assert eta <= {"fp64": 1e-12, "fp32": 1e-5, "bf16upd": 1e-2}[precision]
