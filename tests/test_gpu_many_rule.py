"""Which solves of more than 2^21 rows are launched as workgroups of 1,024
rows (``SolveInfo.shape``: 64-row blocks per wave, workgroups) and which as at
most 1,024 workgroups."""

import pytest
import torch

from paper_1612_01395_amd import solver
from gpu_util import require_gpu

pytestmark = pytest.mark.gpu

C5 = (-1.0, -1.0, 4.5, -1.0, -1.0)
C7 = (-1.0, -1.0, -1.0, 7.0, -1.0, -1.0, -1.0)


def many(op, **kw):
    b = torch.ones(op.n, dtype=torch.float64, device="cuda")
    shape = solver.solve(op, b, maxit=1, tol=0.0, **kw)[1].shape
    if shape[1] > 1024:
        assert shape == (4, -(-op.n // 1024))
    return shape[1] > 1024


def per_row(nx, ny, nz, c):
    n = nx * ny * nz
    coef = torch.tensor(c, dtype=torch.float64, device="cuda").repeat_interleave(n)
    return solver.stencil(nx, ny, nz, coef)


@pytest.fixture(autouse=True)
def no_switches(monkeypatch):
    for k in ("PBCGS_PERSIST", "PBCGS_MANY", "PBCGS_R", "PBCGS_GTARGET", "PBCGS_VALUE_CODES"):
        monkeypatch.delenv(k, raising=False)


def test_five_points():
    """Few vectors and a short row up to 2^22 rows: at most 1,024 workgroups."""
    require_gpu()
    small, large = solver.stencil(1500, 1500, 1, C5), solver.stencil(2100, 2100, 1, C5)
    ops = [small, per_row(1500, 1500, 1, C5)]
    for op in ops:
        for variant, precond, want in (("bicgstab", None, False), ("bicgstab", "jacobi", True), ("cg", None, False),
                                       ("cg", "jacobi", False), ("cgcg", None, False), ("pipe_cg", None, False),
                                       ("pipe_cg", "jacobi", False), ("ca_bicgstab", None, True),
                                       ("pbicgstab_rr", None, False)):
            assert many(op, variant=variant, precond=precond) == want, (op.kind, variant, precond)
    assert not many(small, variant="pbicgstab_rr", precision="fp32_rr64")
    for variant in ("bicgstab", "cg", "pipe_cg", "pbicgstab_rr"):
        assert many(large, variant=variant), variant
    assert many(large, variant="pbicgstab_rr", precision="fp32_rr64")


def test_value_codes():
    require_gpu()
    for n, want in ((1500, True), (1900, False)):
        op = solver.csr(*solver.assemble_convdiff(2, n, 5, (20.0, 10.0)))
        for variant in ("bicgstab", "cg"):
            assert many(op, variant=variant) == want, (n, variant)
        assert many(op, variant="ca_bicgstab")


def test_seven_points():
    require_gpu()
    for n, cg in ((130, True), (150, False)):
        op = solver.stencil(n, n, n, C7)
        for variant, precond, want in (("bicgstab", None, True), ("cg", None, cg), ("cg", "jacobi", cg),
                                       ("cgcg", None, True), ("pipe_cg", None, False), ("pipe_cg", "jacobi", True),
                                       ("pbicgstab_rr", None, False)):
            assert many(op, variant=variant, precond=precond) == want, (n, variant, precond)
        assert many(op, variant="pbicgstab_rr", precision="fp32_rr64")
    assert many(per_row(150, 150, 150, C7), variant="cg")
