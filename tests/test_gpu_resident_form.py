"""Which form a solve runs in (``SolveInfo.resident_rows``): the rows per
thread of the resident launch, or 0 for the streamed kernels."""

import numpy as np
import pytest

from paper_1612_01395_amd import solver
from gpu_util import csr_op, dev_t, host, require_gpu, same, say
from test_gpu_resident import ALG, band

pytestmark = pytest.mark.gpu

SPD = ("cg", "cgcg", "pipe_cg")


@pytest.fixture(autouse=True)
def no_switches(monkeypatch):
    for k in ("PBCGS_PERSIST", "PBCGS_RESIDENT_ROWS", "PBCGS_R", "PBCGS_GTARGET", "PBCGS_BATCH_GCAP", "PBCGS_MANY"):
        monkeypatch.delenv(k, raising=False)


def ran(op, **kw):
    b = dev_t(np.random.default_rng(op.n).standard_normal(op.n))
    return solver.solve(op, b, **dict(dict(tol=1e-9, maxit=5), **kw))[1].resident_rows


@pytest.mark.parametrize("variant", list(ALG))
@pytest.mark.parametrize("K", [2, 4, 8, 16])
def test_forced_rows_per_thread(K, variant, monkeypatch):
    """The rows per thread asked for run, with windows only and with far
    diagonals; 16 of them do not exist with Jacobi as written (but for CG and
    Chronopoulos & Gear CG) nor for varying values, which stream instead."""
    require_gpu()
    rows = 512 * K
    monkeypatch.setenv("PBCGS_RESIDENT_ROWS", str(K))
    for offs in ([-33, -1, 1, 33], [-(rows // 2 + 7), -64, -1, 1, 64, rows // 2 + 7]):
        for varying in (False,) if variant in SPD else (False, True):  # the symmetric band holds one value a diagonal
            op = csr_op(band(2 * rows + 65, offs, varying, spd=variant in SPD))
            for precond in (None, "jacobi") if variant in SPD else (None, "jacobi", "jacobi_folded"):
                want = K
                if K == 16 and (varying or (precond == "jacobi" and variant not in ("cg", "cgcg"))):
                    want = 0
                say(f"form {variant} {precond} K={K} offsets={offs} varying={varying}")
                assert ran(op, variant=variant, precond=precond) == want, (variant, precond, K, offs, varying)


def test_solves_that_stream(monkeypatch):
    """What asks for the streamed kernels gets them, and only that."""
    require_gpu()
    op = solver.stencil(60, 50, 1, (-1.0, -1.25, 4.5, -0.999, -0.75))
    assert ran(op) > 0
    assert ran(op, graph=False) == 0 and ran(op, time_kernels=True) == 0
    assert ran(op, variant="ca_bicgstab") == 0 and ran(op, precision="fp32_rr64") == 0
    A = csr_op(band(3000, [-40, -1, 1, 40], False))
    assert ran(A) > 0
    assert ran(A, index32=True) == 0 and ran(A, diagonal_layout=False) == 0
    for k, v in (("PBCGS_PERSIST", "0"), ("PBCGS_R", "2"), ("PBCGS_MANY", "0")):
        monkeypatch.setenv(k, v)
        assert ran(A) == 0, k
        monkeypatch.delenv(k)
    b = dev_t(np.ones(A.n))
    x = dev_t(np.zeros(A.n))
    assert solver.solve_noalloc(A, b, x, maxit=3)[1].resident_rows == 0


@pytest.mark.parametrize("variant", ["pbicgstab_rr", "bicgstab"])
def test_batches(variant, monkeypatch):
    require_gpu()
    ops = [solver.csr(*solver.assemble_convdiff(2, n, 5, (20.0, 10.0))) for n in (512, 256, 64)]
    bs = [dev_t(np.ones(A.n)) for A in ops]
    kw = dict(variant=variant, maxit=8)
    assert [i.resident_rows for i in solver.solve_batched(ops, bs, **kw)[1]] == [8, 8, 8]
    ops.append(csr_op(band(2000, [-40, -1, 1, 40], True)))
    bs.append(dev_t(np.ones(2000)))
    assert [i.resident_rows for i in solver.solve_batched(ops, bs, **kw)[1]] == [0, 0, 0, 0]
    monkeypatch.setenv("PBCGS_PERSIST", "0")
    assert [i.resident_rows for i in solver.solve_batched(ops[:3], bs[:3], **kw)[1]] == [0, 0, 0]


def test_short_budgets_stream(monkeypatch):
    """A budget too short to pay for what lies beside a resident launch streams, where that is cheaper."""
    require_gpu()
    small = csr_op(band(3000, [-40, -1, 1, 40], False))
    large = solver.stencil(512, 512, 1, (-1.0, -1.25, 4.5, -0.999, -0.75))
    for variant in ALG:
        assert [ran(small, variant=variant, maxit=m) > 0 for m in (0, 1, 2)] == [False, False, True], variant
        assert ran(large, variant=variant, maxit=0) > 0, variant
    ops, bs = [small] * 3, [dev_t(np.ones(3000))] * 3
    for m in (0, 7, 8):
        assert {i.resident_rows > 0 for i in solver.solve_batched(ops, bs, maxit=m)[1]} == {m == 8}, m
    monkeypatch.setenv("PBCGS_PERSIST", "1")
    assert ran(small, maxit=0) > 0 and solver.solve_batched(ops, bs, maxit=0)[1][0].resident_rows > 0


def test_budgets_one_launch_may_hold():
    """Budgets above 200,000 iterations stream: a launch cannot be interrupted."""
    require_gpu()
    op = csr_op(band(3000, [-40, -1, 1, 40], False))
    for variant in ALG:
        assert [ran(op, variant=variant, maxit=m) > 0 for m in (200000, 200001)] == [True, False], variant
    ops, bs = [op] * 3, [dev_t(np.ones(3000))] * 3
    for m in (200000, 200001):
        assert {i.resident_rows > 0 for i in solver.solve_batched(ops, bs, maxit=m)[1]} == {m == 200000}, m


def test_surroundings_a_window_may_hold():
    """Inner diagonals up to 3,584 rows away; the results are the streamed ones."""
    require_gpu()
    n = 40000
    b = dev_t(np.random.default_rng(6).standard_normal(n))
    for H, want in ((3072, True), (3584, True), (3586, False)):
        for values in (False, True):
            op = csr_op(band(n, [-H - 900, -H, -1, 1, H, H + 900], values))
            say(f"window H={H} varying={values}")
            for variant in ("pbicgstab", "bicgstab"):
                kw = dict(variant=variant, tol=0.0, maxit=6, history=True)
                x, i = solver.solve(op, b, **kw)
                y, s = solver.solve(op, b, graph=False, **kw)
                assert (i.resident_rows > 0) == want, (H, values, variant)
                assert same(host(x), host(y)) and same(host(i.history), host(s.history)), (H, values, variant)
