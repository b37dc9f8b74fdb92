"""Shapes whose products with M + G have 64 to 127 tiles of 256 x 256: all of them split over the contraction on the
direct-load path."""
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, one_step_report
from test_gpu_double import run as run_double
from test_gpu_lazy import run_lazy
from test_gpu_transposed import T, run as run_transposed

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA


@pytest.mark.parametrize("shape", [(4096, 4352, 1024), (5120, 4096, 1024)])
def test_two_steps(shape):
    gp = GpuProblem([shape], True, "bf16")
    for t in range(2):
        g = gp.grads_np(t)[0]
        x_in, m_in, q_in = gp.host()
        gp.upload_grads([g])
        assert gp.step(MU, ETA) == (0, -1), (shape, t)
        rep, _ = one_step_report(gp, 0, x_in, m_in, q_in, gp.grad_as_f32(g, True), MU, ETA, "lapack")
        # the bounds of the fixed-shape parity tests in this mode
        assert rep["X"] <= 2e-2 and rep["M"] <= 2e-2 and rep["dX"] <= 4e-2 and rep["dM"] <= 4e-2, (shape, t, rep)
        assert rep["orth"] <= 1e-3, (shape, t, rep)


# the other steps on the same route, the bounds being those of their own tests on the direct-load path
def test_lazy_with_and_without_a_refresh():
    run_lazy([(4096, 4352, 1024)], True, "bf16", 2, 2, 2e-2, 2e-4, method="lapack")


def test_transposed_form():
    run_transposed([(4352, 4096, 1024)], [T], True, "bf16", 2, 2e-2, method="lapack")


@pytest.mark.parametrize("warm", [True, False])
def test_double_dion(warm):
    # (from an empty buffer the second stage is badly conditioned while it fills up: the wider bound of the test at 8192 x 8192)
    run_double([(4096, 4352)], 256, 1024, True, "bf16", 2, 2e-2, method="lapack", warm=warm, dx_tol=None if warm else 0.15)
