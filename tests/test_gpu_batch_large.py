"""Batches of very many systems, in the resident form and streamed: the same
bits, no limit of the launch grid in the way and no more memory than the
streamed batch."""

import numpy as np
import pytest
import torch

import oracle

from paper_1612_01395_amd import solver
from gpu_util import csr_op, dev_t, host, require_gpu, same, say

pytestmark = pytest.mark.gpu

ALG = {"bicgstab": oracle.ALG_BICGSTAB, "pbicgstab_rr": oracle.ALG_PBICGSTAB_RR}


def tridiagonal(n, ctx):
    i = np.arange(n)
    rows = np.concatenate([i, i[1:], i[:-1]])
    cols = np.concatenate([i, i[1:] - 1, i[:-1] + 1])
    vals = np.concatenate([np.full(n, 3.0), np.full(n - 1, -1.0), np.full(n - 1, -1.25)])
    order = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, np.int32)
    np.add.at(rp, rows + 1, 1)
    t = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
         for a in (np.cumsum(rp).astype(np.int32), cols[order].astype(np.int32), vals[order])]
    return solver.csr(*t, ctx=ctx)


@pytest.mark.parametrize("variant", ["pbicgstab_rr", "bicgstab"])
def test_more_systems_than_a_grid_has_rows(variant, monkeypatch):
    """66,000 systems: more than the 65,536 a launch takes in its second grid dimension."""
    require_gpu()
    count, n = 66000, 5
    ctx = solver.Context()
    A = tridiagonal(n, ctx)
    g = torch.Generator(device="cuda").manual_seed(1)
    b = torch.randn(count, n, dtype=torch.float64, device="cuda", generator=g)
    out = []
    for mode in ("1", "0"):
        monkeypatch.setenv("PBCGS_PERSIST", mode)
        x = torch.empty_like(b)
        say(f"batch of {count} {variant} mode {mode}")
        _, infos = solver.solve_batched([A] * count, list(b.unbind(0)), outs=list(x.unbind(0)), variant=variant,
                                        maxit=4, rr_period=2)
        out.append((x.cpu().numpy(), [(i.iters, i.n_rr, i.status, i.relres_rec, i.relres_true) for i in infos]))
        assert {i.resident_rows > 0 for i in infos} == {mode == "1"}
    (x, i), (y, k) = out
    assert same(x, y) and i == k


def test_memory_of_many_small_systems(monkeypatch):
    """3,000 systems of 100 rows take no more device memory in the resident
    form than streamed, beyond what 300 of them take (a queue's first launch
    of a kernel allocates that kernel's scratch, whatever the batch)."""
    require_gpu()
    used = []
    for mode in ("0", "1"):
        monkeypatch.setenv("PBCGS_PERSIST", mode)
        ctx = solver.Context()
        A = tridiagonal(100, ctx)
        b = torch.ones(3000, 100, dtype=torch.float64, device="cuda")
        x = torch.empty_like(b)
        bs, outs = list(b.unbind(0)), list(x.unbind(0))
        solver.solve_batched([A] * 300, bs[:300], outs=outs[:300], maxit=3)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        solver.solve_batched([A] * 3000, bs, outs=outs, maxit=3)
        used.append(before - torch.cuda.mem_get_info()[0])
    say(f"bytes taken: streamed {used[0]}, resident {used[1]}")
    assert used[1] <= used[0] + (4 << 20)


def test_which_batches_stream():
    """Many small systems stream, where a workgroup of the resident form would
    be mostly empty; batches that one launch holds, and larger systems, do not.
    The leftover systems' bits are the streamed ones."""
    require_gpu()
    ctx = solver.Context()
    for n, count, resident in ((100, 300, False), (100, 200, True), (2000, 300, True)):
        A = tridiagonal(n, ctx)
        g = torch.Generator(device="cuda").manual_seed(n)
        b = torch.randn(count, n, dtype=torch.float64, device="cuda", generator=g)
        out = []
        for graph in (True, False):  # the second: streamed
            x = torch.empty_like(b)
            _, infos = solver.solve_batched([A] * count, list(b.unbind(0)), outs=list(x.unbind(0)), maxit=12,
                                            rr_period=5, graph=graph)
            assert {i.resident_rows > 0 for i in infos} == {resident and graph}, (n, count, graph)
            out.append((x.cpu().numpy(), [(i.iters, i.n_rr, i.status, i.relres_rec, i.relres_true) for i in infos]))
        assert same(out[0][0], out[1][0]) and out[0][1] == out[1][1], (n, count)


@pytest.mark.parametrize("variant", list(ALG))
@pytest.mark.parametrize("diagonals", [7, 8, 27, 32])
def test_layouts_of_many_diagonals(diagonals, variant):
    """Layouts of more than seven diagonals have no place in the resident
    form's tables: such a batch streams, whatever stands beside them."""
    require_gpu()
    rng = np.random.default_rng(diagonals)
    n = 2000
    offs = np.sort(np.concatenate([[0], 1 + rng.choice(120, diagonals - 1, replace=False)]))
    rows, cols, vals = [], [], []
    for o in offs:
        r = np.arange(n - o)
        rows.append(r)
        cols.append(r + o)
        vals.append(np.full(r.size, 40.0 if o == 0 else -0.5))
    r, c, v = (np.concatenate(a) for a in (rows, cols, vals))
    order = np.lexsort((c, r))
    wide = oracle.CSR(np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32),
                      c[order].astype(np.int32), v[order])
    grid = oracle.assemble(2, 20, 5, (20.0, 10.0))
    As = [grid, wide, grid]
    ops = [csr_op(A) for A in As]
    assert ops[1].diagonals == diagonals
    bs = [rng.standard_normal(A.n) for A in As]
    kw = dict(tol=1e-9, maxit=30, rr_period=7)
    xs, infos = solver.solve_batched(ops, [dev_t(b) for b in bs], variant=variant, **kw)
    for A, b, x, info in zip(As, bs, xs, infos):
        x_or, i_or = oracle.solve(A, b, algo=ALG[variant], **kw)
        assert (info.resident_rows > 0) == (diagonals <= 7)
        assert (info.status, info.iters, info.n_rr) == (i_or["status"], i_or["iters"], i_or["n_rr"])
        assert same(host(x), x_or)
