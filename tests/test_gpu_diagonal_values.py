"""How many values the diagonals of a large CSR operator hold decides the form
its solves take: one value each, the resident form; at most sixteen, the value
codes; more, the layout's values.  The library looks at a few rows before all
of them, so the values vary everywhere, only at the ends or in one entry here;
the results are the streamed form's bit for bit, and so is what it says of the
codes."""

import numpy as np
import pytest

import oracle
from paper_1612_01395_amd import solver
from gpu_util import csr_op, dev_t, host, require_gpu, same, say
from test_gpu_resident import band

pytestmark = pytest.mark.gpu

N = 263001  # above 2^18
A0 = band(N, [-500, -1, 1, 500], varying=False)
ROW = np.repeat(np.arange(N), np.diff(A0.row_ptr))
WHERE = {"everywhere": np.ones(ROW.size, bool), "first rows": ROW < 3000, "last rows": ROW >= N - 70,
         "main diagonal": ROW == A0.col, "one entry": np.arange(ROW.size) == ROW.size - 5}


@pytest.mark.parametrize("where", list(WHERE))
@pytest.mark.parametrize("k", [1, 2, 16, 17, 18, 19, 200])
def test_forms(k, where, monkeypatch):
    """k values per diagonal: in turn over the rows chosen."""
    require_gpu()
    for name in ("PBCGS_PERSIST", "PBCGS_VALUE_CODES"):
        monkeypatch.delenv(name, raising=False)
    v = A0.val.copy()
    pick = WHERE[where]
    v[pick] *= 1.0 + 2.0 ** -12 * (ROW[pick] % k)
    distinct = max(np.unique(v[ROW + d == A0.col]).size for d in (-500, -1, 0, 1, 500))
    op = csr_op(oracle.CSR(A0.row_ptr, A0.col, v))
    b = dev_t(np.random.default_rng(k).standard_normal(N))
    for variant, precond in (("pbicgstab_rr", None), ("bicgstab", "jacobi"), ("pbicgstab_rr", "jacobi_folded")):
        out = []
        for mode in (None, "0"):
            if mode:
                monkeypatch.setenv("PBCGS_PERSIST", mode)
            out.append(solver.solve(op, b, variant=variant, precond=precond, tol=0.0, maxit=6, rr_period=4))
            monkeypatch.delenv("PBCGS_PERSIST", raising=False)
        (x, i), (y, s) = out
        say(f"values k={k} {where} {variant} {precond}: {distinct} values, resident {i.resident_rows}, "
            f"codes {i.value_codes}")
        assert same(host(x), host(y)) and (i.iters, i.status, i.n_rr) == (s.iters, s.status, s.n_rr)
        assert i.value_codes == s.value_codes and s.resident_rows == 0
        if precond is None:
            assert (i.resident_rows > 0) == (distinct == 1) and i.value_codes == (distinct <= 16)
