"""Launches of more than 1,024 small workgroups with folded partial sums
against launches of at most 1,024: the same bits for every method, the
binary32 form and each kind of operator, at row counts around a whole fold of
1,024 partial sums."""

import pytest
import torch

from paper_1612_01395_amd import solver
from gpu_util import dev_t, host, require_gpu, same, say

pytestmark = pytest.mark.gpu


def both(op, monkeypatch, R, seed=0, **kw):
    g = torch.Generator(device="cuda").manual_seed(seed)
    b = torch.randn(op.n, dtype=torch.float64, device="cuda", generator=g)
    monkeypatch.setenv("PBCGS_PERSIST", "0")
    out = []
    for many in ("0", str(R)):
        monkeypatch.setenv("PBCGS_MANY", many)
        out.append(solver.solve(op, b, history=True, tol=0.0, maxit=9, rr_period=4, **kw))
    (x, i), (y, k) = out
    assert i.shape[1] <= 1024 < k.shape[1] and k.shape[0] == R, (i.shape, k.shape)
    assert (i.status, i.iters, i.n_rr) == (k.status, k.iters, k.n_rr), kw
    assert same(host(x), host(y)) and same(host(i.history), host(k.history)), kw
    assert same([i.relres_rec, i.relres_true], [k.relres_rec, k.relres_true]), kw


@pytest.mark.parametrize("variant", ["pbicgstab_rr", "pbicgstab", "bicgstab", "ca_bicgstab", "cg", "cgcg", "pipe_cg"])
def test_methods(variant, monkeypatch):
    require_gpu()
    for extra in (1, 512 * 1024 - 1, 512 * 1024 + 3):  # one partial past a fold, one short of two, one past two
        n = 512 * 1024 + extra
        op = solver.stencil(n, 1, 1, (-1.0, -1.0, 4.0, -1.0, -1.0))
        for precond in ((None,) if variant == "ca_bicgstab" else (None, "jacobi")):
            say(f"many workgroups {variant} {precond} n={n}")
            both(op, monkeypatch, 2, variant=variant, precond=precond)


@pytest.mark.parametrize("kind", ["layout", "csr", "conv27", "binary32"])
def test_operators(kind, monkeypatch):
    require_gpu()
    if kind in ("conv27", "csr"):
        n = 85
        kappa = dev_t(__import__("numpy").random.default_rng(1).random((n + 1) ** 3) + 0.5)
        if kind == "conv27":
            op = solver.convdiff27(n, kappa, (10.0, 0.0, 5.0), 0.1)
        else:
            op = solver.csr(*solver.assemble_convdiff(3, n, 27, (10.0, 0.0, 5.0), kappa=kappa, shift=0.1))
    else:
        op = solver.csr(*solver.assemble_convdiff(3, 103, 7, (5.0, 3.0, 1.0)))
    kw = dict(variant="pbicgstab_rr", precond="jacobi_folded")
    if kind == "binary32":
        kw["precision"] = "fp32_rr64"
    if kind == "csr":
        kw["diagonal_layout"] = False
    for R in (1, 2, 4) if op.n > 1024 * 1024 else (1, 2):
        both(op, monkeypatch, R, seed=R, **kw)
