"""Resident solves (one cooperative launch, Krylov vectors in registers and
LDS) against the oracle, bit for bit: every method and preconditioner form at
each number of rows per thread, row counts around the workgroup's 512 K rows,
diagonals read from the windows and from the exchange buffers, one value per
diagonal and varying values, and the forms a solve must not take.

The tolerance is zero: sums run in the same pairwise order as the oracle's.
"""

import numpy as np
import pytest

import oracle
from paper_1612_01395_amd import solver
from gpu_util import csr_op, dev_t, host, require_gpu, same, say

pytestmark = pytest.mark.gpu

ALG = {"bicgstab": oracle.ALG_BICGSTAB, "pbicgstab": oracle.ALG_PBICGSTAB, "pbicgstab_rr": oracle.ALG_PBICGSTAB_RR,
       "cg": oracle.ALG_CG, "cgcg": oracle.ALG_CGCG, "pipe_cg": oracle.ALG_PIPE_CG}
KW = dict(tol=1e-9, maxit=23, rr_period=6)


def band(n, offs, varying, spd=False, seed=0):
    """A banded matrix of the given off-diagonal offsets plus the main one,
    dominant, with every fifth row missing its first off-diagonal."""
    rng = np.random.default_rng([n, seed])
    rows, cols, vals = [], [], []
    i = np.arange(n)
    offs = sorted(set(offs) | {0})
    for k, o in enumerate(offs):
        r = i[(i + o >= 0) & (i + o < n)]
        if k == 0 and not spd and len(offs) > 1:
            r = r[r % 5 != 3]
        if o == 0:
            v = np.full(r.size, 2.0 * len(offs)) + (rng.random(r.size) if varying else 0.0)
        elif spd:
            v = np.full(r.size, -1.0)
        else:
            v = -rng.random(r.size) if varying else np.full(r.size, -0.25 - 0.125 * k)
        rows.append(r)
        cols.append(r + o)
        vals.append(v)
    r, c, v = (np.concatenate(a) for a in (rows, cols, vals))
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, r + 1, 1)
    return oracle.CSR(np.cumsum(rp).astype(np.int32), c[order].astype(np.int32), v[order])


def check(A, op, variant, precond, K, monkeypatch, x0=None, **extra):
    kw = dict(KW, **extra)
    rng = np.random.default_rng(A.n)
    b = rng.standard_normal(A.n)
    d = oracle.jacobi_dinv(A) if precond else None
    solve = oracle.solve_folded if precond == "jacobi_folded" else oracle.solve
    x_or, i_or = solve(A, b, algo=ALG[variant], dinv=d, x0=x0, history=True, **kw)
    monkeypatch.setenv("PBCGS_PERSIST", "1")
    monkeypatch.setenv("PBCGS_RESIDENT_ROWS", str(K))
    x, info = solver.solve(op, dev_t(b), None if x0 is None else dev_t(x0), variant=variant, precond=precond,
                           history=True, **kw)
    what = (A.n, variant, precond, K)
    assert (info.status, info.iters, info.n_rr) == (i_or["status"], i_or["iters"], i_or["n_rr"]), (what, info, i_or)
    assert same(host(x), x_or), what
    assert same([info.relres_rec, info.relres_true], [i_or["relres_rec"], i_or["relres_true"]]), what
    assert same(host(info.history), i_or["history"]), what


@pytest.mark.parametrize("variant", list(ALG))
@pytest.mark.parametrize("K", [2, 4, 8, 16])
def test_rows_around_a_workgroup(K, variant, monkeypatch):
    """Row counts one below, at and one above whole workgroups, near and far diagonals, each Jacobi form."""
    require_gpu()
    rows = 512 * K
    spd = variant in ("cg", "cgcg", "pipe_cg")
    sizes = [rows + 1, 2 * rows - 1, 2 * rows, 3 * rows + 65] + ([1, 2, 127, rows] if K <= 8 else [])
    for n in sizes:
        for offs in ([-33, -1, 1, 33], [-(rows // 2 + 7), -64, -1, 1, 64, rows // 2 + 7]):
            offs = [o for o in offs if abs(o) < n]
            A = band(n, offs, varying=False, spd=spd)
            op = csr_op(A)
            forms = [None, "jacobi"] if spd else [None, "jacobi", "jacobi_folded"]
            for precond in forms:
                say(f"resident {variant} {precond} K={K} n={n} offsets={offs}")
                check(A, op, variant, precond, K, monkeypatch)


@pytest.mark.parametrize("variant", list(ALG))
@pytest.mark.parametrize("K", [2, 4, 8])
def test_varying_values_and_x0(K, variant, monkeypatch):
    """Values that vary along a diagonal (read from the layout), a Jacobi vector, x_0, odd offsets on both sides only."""
    require_gpu()
    spd = variant in ("cg", "cgcg", "pipe_cg")
    n = 1024 * K + 77
    for offs in ([-3, 5], [-(256 * K + 9), -1, 1, 256 * K + 9]):
        A = band(n, offs if not spd else [-o for o in offs[-1:]] + offs[-1:], varying=not spd, spd=spd)
        if spd:  # a varying diagonal only
            v = A.val.copy()
            diag = np.repeat(np.arange(n), np.diff(A.row_ptr)) == A.col
            v[diag] += np.random.default_rng(1).random(n)
            A = oracle.CSR(A.row_ptr, A.col, v)
        op = csr_op(A)
        x0 = np.random.default_rng(2).standard_normal(n)
        for precond in ([None, "jacobi"] if spd else [None, "jacobi", "jacobi_folded"]):
            say(f"resident varying {variant} {precond} K={K} offsets={offs}")
            check(A, op, variant, precond, K, monkeypatch, x0=x0)


@pytest.mark.parametrize("variant", list(ALG))
def test_limits_and_statuses(variant, monkeypatch):
    """maxit 0 and 1, replacement in every iteration, b = 0, NaN and Inf in b."""
    require_gpu()
    A = band(3000, [-40, -1, 1, 40], varying=False, spd=True)
    op = csr_op(A)
    for kw in (dict(maxit=0), dict(maxit=1, tol=0.0), dict(rr_period=1), dict(rr_period=2, rr_max=3), dict(tol=0.0)):
        check(A, op, variant, None, 2, monkeypatch, **kw)
    for bad in (0.0, np.nan, np.inf):
        b = np.zeros(A.n)
        b[1234] = bad
        x_or, i_or = oracle.solve(A, b, algo=ALG[variant], **KW)
        x, info = solver.solve(op, dev_t(b), variant=variant, **KW)
        assert (info.status, info.iters) == (i_or["status"], i_or["iters"]), (variant, bad)
        assert same(host(x), x_or), (variant, bad)


def test_same_bits_as_the_streamed_kernels_by_default(monkeypatch):
    """The launch the library chooses by itself on grids of one to 256
    workgroups against the streamed kernels, stencil and CSR."""
    require_gpu()
    for k in ("PBCGS_RESIDENT_ROWS", "PBCGS_PERSIST"):
        monkeypatch.delenv(k, raising=False)
    for dims in ((17, 1, 1), (70, 33, 1), (41, 41, 41), (127, 64, 64), (100, 100, 99)):
        nx, ny, nz = dims
        coef = (-1.0, -1.25, 4.5, -0.999, -0.75) if nz == 1 else (-1.0, -1.5, -1.25, 7.0, -1.0, -0.75, -0.5)
        op = solver.stencil(nx, ny, nz, coef)
        b = dev_t(np.random.default_rng(3).standard_normal(op.n))
        for variant in ("pbicgstab_rr", "bicgstab"):
            x, info = solver.solve(op, b, variant=variant, maxit=60, rr_period=25, history=True)
            y, ref = solver.solve(op, b, variant=variant, maxit=60, rr_period=25, history=True, graph=False)
            assert (info.iters, info.n_rr, info.status) == (ref.iters, ref.n_rr, ref.status), (dims, variant)
            assert same(host(x), host(y)) and same(host(info.history), host(ref.history)), (dims, variant)
            assert same([info.relres_rec, info.relres_true], [ref.relres_rec, ref.relres_true]), (dims, variant)


@pytest.mark.parametrize("variant", ["pbicgstab_rr", "bicgstab"])
def test_batch_over_several_launches(variant, monkeypatch):
    """A batch of more workgroups than one launch holds, five and seven
    diagonals together, one to 64 workgroups a system; then with one system
    whose values vary, which takes the streamed kernels."""
    require_gpu()
    for k in ("PBCGS_RESIDENT_ROWS", "PBCGS_BATCH_GCAP"):
        monkeypatch.delenv(k, raising=False)
    ops, bs = [], []
    for n in (512, 500, 333, 64, 65, 1, 2, 400, 90, 511, 128, 300):
        ops.append(solver.csr(*solver.assemble_convdiff(2, n, 5, (20.0, 10.0))))
    for n in (30, 3, 17):
        ops.append(solver.csr(*solver.assemble_convdiff(3, n, 7, (50.0, 30.0, 10.0))))
    rng = np.random.default_rng(8)
    kw = dict(variant=variant, tol=1e-9, maxit=45, rr_period=20)
    for varying in (False, True):
        if varying:
            ops.append(csr_op(band(2000, [-40, -1, 1, 40], varying=True)))
        bs = [dev_t(rng.standard_normal(A.n)) for A in ops]
        out = []
        for mode in ("0", "1"):
            monkeypatch.setenv("PBCGS_PERSIST", mode)
            out.append(solver.solve_batched(ops, bs, **kw))
        (xs, si), (ys, ti) = out
        for k, (x, y, i, t) in enumerate(zip(xs, ys, si, ti)):
            assert (i.iters, i.n_rr, i.status) == (t.iters, t.n_rr, t.status), (k, i, t)
            assert same(host(x), host(y)) and same([i.relres_rec, i.relres_true], [t.relres_rec, t.relres_true]), k
