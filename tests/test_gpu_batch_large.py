"""Batches of very many systems, in the resident form and streamed: the same
bits, no limit of the launch grid in the way and no more memory than the
streamed batch."""

import numpy as np
import pytest
import torch

from paper_1612_01395_amd import solver
from gpu_util import require_gpu, same, say

pytestmark = pytest.mark.gpu


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
