"""A resident launch whose waits time out: the workgroups leave, the caller's x
is untouched and the solve starts again in the streamed kernels, with their
bits.  PBCGS_RESIDENT_GIVE_UP=1 makes the workgroups wait for one that is not
there, so that the bounded wait ends by itself after about 0.07 s; =2 counts
a solve that ran to its end as timed out.  Contexts of their own: one that gave
up streams for a while.
"""

import numpy as np
import pytest

from paper_1612_01395_amd import solver
from gpu_util import dev_t, host, require_gpu, same, say
from test_gpu_resident import ALG, band

pytestmark = pytest.mark.gpu

N = 9000
SPD = ("cg", "cgcg", "pipe_cg")


@pytest.mark.parametrize("variant", list(ALG))
def test_single(variant, monkeypatch):
    require_gpu()
    monkeypatch.setenv("PBCGS_RESIDENT_ROWS", "2")  # several workgroups
    spd = variant in SPD
    ctx = solver.Context()
    rng = np.random.default_rng(4)
    b, x0 = dev_t(rng.standard_normal(N)), dev_t(rng.standard_normal(N))
    for varying in (False,) if spd else (False, True):
        A = band(N, [-700, -1, 1, 700], varying, spd=spd)
        op = solver.csr(dev_t(A.row_ptr), dev_t(A.col), dev_t(A.val), ctx=ctx)
        for precond in (None, "jacobi") if spd else (None, "jacobi", "jacobi_folded"):
            kw = dict(variant=variant, precond=precond, tol=0.0, maxit=20, rr_period=6, history=True)
            monkeypatch.setenv("PBCGS_PERSIST", "0")
            y, ref = solver.solve(op, b, x0, **kw)
            monkeypatch.setenv("PBCGS_PERSIST", "1")
            assert solver.solve(op, b, x0, **kw)[1].resident_rows == 2
            # the real wait once per method, with the most state to give up
            for e in (1, 2) if precond == "jacobi" and varying == (not spd) else (2,):
                say(f"give up {variant} {precond} varying={varying} form {e}")
                monkeypatch.setenv("PBCGS_RESIDENT_GIVE_UP", str(e))
                x, info = solver.solve(op, b, x0, **kw)
                monkeypatch.delenv("PBCGS_RESIDENT_GIVE_UP")
                assert info.resident_rows == 0
                assert (info.iters, info.n_rr, info.status) == (ref.iters, ref.n_rr, ref.status)
                assert same(host(x), host(y)) and same(host(info.history), host(ref.history))
                assert same([info.relres_rec, info.relres_true], [ref.relres_rec, ref.relres_true])


@pytest.mark.parametrize("variant", ["pbicgstab_rr", "bicgstab"])
def test_batch(variant, monkeypatch):
    """Systems of one workgroup, which exchange nothing, beside larger ones that give up."""
    require_gpu()
    ctx = solver.Context()
    ops = [solver.csr(*solver.assemble_convdiff(2, n, 5, (20.0, 10.0), ctx=ctx), ctx=ctx) for n in (300, 20, 100, 3, 64)]
    rng = np.random.default_rng(5)
    bs, x0s = ([dev_t(rng.standard_normal(A.n)) for A in ops] for _ in range(2))
    kw = dict(variant=variant, tol=0.0, maxit=20, rr_period=6)
    monkeypatch.setenv("PBCGS_PERSIST", "0")
    ys, refs = solver.solve_batched(ops, bs, x0s, **kw)
    monkeypatch.setenv("PBCGS_PERSIST", "1")
    for e in (1, 2):
        say(f"give up batch {variant} form {e}")
        monkeypatch.setenv("PBCGS_RESIDENT_GIVE_UP", str(e))
        xs, infos = solver.solve_batched(ops, bs, x0s, **kw)
        for x, y, i, r in zip(xs, ys, infos, refs):
            assert i.resident_rows == 0
            assert (i.iters, i.n_rr, i.status) == (r.iters, r.n_rr, r.status)
            assert same(host(x), host(y)) and same([i.relres_rec, i.relres_true], [r.relres_rec, r.relres_true])


def test_the_next_solves_stream(monkeypatch):
    """After giving up a context streams its next 16 solves, 32 when it gives
    up again at once, 16 again after one that ran to its end; others are not
    concerned."""
    require_gpu()
    for k in ("PBCGS_PERSIST", "PBCGS_RESIDENT_ROWS"):
        monkeypatch.delenv(k, raising=False)
    ctx, other = solver.Context(), solver.Context()
    coef = (-1.0, -1.25, 4.5, -0.999, -0.75)
    A, B = (solver.stencil(120, 100, 1, coef, ctx=c) for c in (ctx, other))
    b = dev_t(np.ones(A.n))

    def form(op):
        return solver.solve(op, b, maxit=3)[1].resident_rows > 0

    def give_up():
        monkeypatch.setenv("PBCGS_RESIDENT_GIVE_UP", "2")
        assert not form(A)
        monkeypatch.delenv("PBCGS_RESIDENT_GIVE_UP")

    assert form(A) and form(B)
    give_up()
    assert [form(A) for _ in range(16)] == [False] * 16 and form(B)
    give_up()
    assert [form(A) for _ in range(32)] == [False] * 32
    assert form(A)
    give_up()
    assert [form(A) for _ in range(17)] == [False] * 16 + [True]
