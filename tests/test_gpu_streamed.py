"""The streamed kernels on systems small enough for the resident form: the
parity, chunking, launch-shape, batch and poisoning tests again with the
resident form switched off, so that the graph-launched layout and stencil
kernels, their polling and their tuned shapes are the ones that run."""

import pytest
import torch

from paper_1612_01395_amd import solver
from gpu_util import require_gpu

# collected here again, under the fixture below
from test_gpu_adjoint import test_adjoint_solve_and_gradient_bitwise  # noqa: F401
from test_gpu_alpha_eq5 import test_eq5_batched_bitwise, test_eq5_bitwise_csr, test_eq5_bitwise_stencil  # noqa: F401
from test_gpu_batched import (test_batched_diagonal_layout, test_batched_equals_individual_oracle_solves,  # noqa: F401
                              test_batched_x0_maxit_and_shapes)
from test_gpu_cg import (test_cg_family_bitwise_csr, test_cg_family_bitwise_stencil,  # noqa: F401
                         test_cg_family_maxit_x0_chunks_and_shapes, test_cg_family_status_cases)
from test_gpu_debug_hooks import (test_poisoned_batched, test_poisoned_bicgstab_family,  # noqa: F401
                                  test_poisoned_cg_family)
from test_gpu_parity import (test_folded_with_x0_and_repeated_calls, test_launch_modes_and_shapes_identical,  # noqa: F401
                             test_rr_max_and_maxit_and_x0, test_solve_bitwise_csr, test_solve_bitwise_stencil,
                             test_solve_bitwise_vector_jacobi, test_status_cases_match_oracle)
from test_gpu_random import test_random_system_bitwise  # noqa: F401
from test_gpu_tune import test_tune_cache_serves_new_operators  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def streamed(monkeypatch):
    monkeypatch.setenv("PBCGS_PERSIST", "0")


def test_the_streamed_form_runs():
    require_gpu()
    op = solver.stencil(50, 40, 1, (-1.0, -1.25, 4.5, -0.999, -0.75))
    b = torch.ones(op.n, dtype=torch.float64, device="cuda")
    assert solver.solve(op, b, maxit=5)[1].resident_rows == 0
