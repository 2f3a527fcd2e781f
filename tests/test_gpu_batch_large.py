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
    """66,000 systems: more than the 65,535 a launch takes in its second grid dimension."""
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
    """3,000 systems of 100 rows take no more device memory in the resident form than streamed."""
    require_gpu()
    used = []
    for mode in ("0", "1"):
        monkeypatch.setenv("PBCGS_PERSIST", mode)
        ctx = solver.Context()
        A = tridiagonal(100, ctx)
        b = torch.ones(3000, 100, dtype=torch.float64, device="cuda")
        x = torch.empty_like(b)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        solver.solve_batched([A] * 3000, list(b.unbind(0)), outs=list(x.unbind(0)), maxit=3)
        used.append(before - torch.cuda.mem_get_info()[0])
    say(f"bytes taken: streamed {used[0]}, resident {used[1]}")
    assert used[1] <= used[0] + (4 << 20)
