"""The update of matrices of any size on the direct-load core beyond test_gpu_ragged_update.py: rows on whole cache lines, with the
streaming hint and without, and the other steps that end in it: the sketch of Double Dion, the transposed form, Lazy-Dion
without refresh.  Nothing is written beside the matrices."""
import numpy as np
import pytest
import torch

from oracle import dion_oracle as orc
from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, relf
from test_gpu_double import DoubleProblem, oracle_with_gpu_decisions
from test_gpu_ragged_update import guarded, guards_intact, test_edges as check_edges
from test_gpu_transposed import T, transposed_report

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA
TOL = 2e-2   # the bound of the fixed-shape parity tests in bf16 mode


# n a multiple of 32: 271 MB of M, X and G without the hint, 520 MB with it (7001 x 4128), whole columns of tiles and the last one
# half; r = 72; then either side of the least rank of rows on 16 bytes
@pytest.mark.parametrize("shape", [(5003, 3008, 360), (4096, 4096, 300), (7001, 4128, 260), (7300, 4608, 72), (6149, 6160, 99), (6149, 6160, 100)])
@pytest.mark.parametrize("g_bf16", [False, True])
def test_rows_on_whole_lines(shape, g_bf16):
    check_edges(shape, g_bf16)


def test_sketch_of_double_dion():
    m, n, r1, r2 = 5003, 2999, 360, 24
    dp = DoubleProblem([(m, n)], r1, r2, True, "bf16")
    flats = []
    for bufs in (dp.D, dp.M1, dp.X):
        flat, bufs[0] = guarded(bufs[0])
        flats.append(flat)
    g = inputs.gradient(m, n, 0, 0, 0, bf16=True)
    dp.upload([g])
    x, m1, v1, m2, v2 = dp.host(0)
    assert dp.step() == ((0, -1), (0, -1))
    assert all(guards_intact(f) for f in flats)
    ref = oracle_with_gpu_decisions(dp, 0, x, inputs.bf16_bits_to_f32(g), m1, v1, m2, v2, "lapack")
    X, M1, V1, M2, V2 = dp.host(0)
    D = dp.D[0].cpu().numpy()
    for a, b in ((X, ref["X"]), (M1, ref["M1"]), (M2, ref["M2"]), (D, ref["D"])):
        assert relf(a, b) <= TOL and relf(a[-1], b[-1]) <= TOL and relf(a[:, -1], b[:, -1]) <= TOL
    assert relf(X.astype(np.float64) - x, ref["X"] - x) <= 3 * TOL


@pytest.mark.parametrize("shape", [(5003, 2999, 360), (4160, 4128, 300)])
def test_transposed_form(shape):
    gp = GpuProblem([shape], True, "bf16", seed=8, forms=[T])
    fx, gp.X[0] = guarded(gp.X[0])
    fm, gp.M[0] = guarded(gp.M[0])
    g = gp.grads_np(0)[0]
    gp.upload_grads([g])
    before = gp.host()
    assert gp.step(MU, ETA) == (0, -1)
    assert guards_intact(fx) and guards_intact(fm)
    rep = transposed_report(gp, 0, *before, gp.grad_as_f32(g, True), "lapack")
    assert rep["vdot"] > 1 - 10 * TOL and rep["vnorm"] < 1e-5, rep
    assert rep["X"] <= TOL and rep["M"] <= TOL and rep["dX"] <= 3 * TOL and rep["dM"] <= 3 * TOL, rep


@pytest.mark.parametrize("shape", [(5003, 2999, 360), (7001, 4128, 260)])
def test_lazy_without_refresh(shape):
    m, n, r = shape
    q = np.linalg.qr(inputs.right_factor_raw(n, r, 5, 0).astype(np.float64))[0].astype(np.float32)
    gp = GpuProblem([shape], True, "bf16", seed=9, q_raw=[q])
    fx, gp.X[0] = guarded(gp.X[0])
    fm, gp.M[0] = guarded(gp.M[0])
    for t in range(2):
        g = gp.grads_np(t)[0]
        x_in, m_in, q_in = gp.host()
        gp.upload_grads([g])
        assert gp.lazy_step(MU, ETA, False) == (0, -1)
        assert guards_intact(fx) and guards_intact(fm)
        ref = orc.lazy_dion_step(x_in, gp.grad_as_f32(g, True), m_in, q_in, MU, ETA, False, "lapack")
        X, M, Q = gp.host()
        assert np.array_equal(Q, q_in)
        assert relf(X, ref["X"]) <= TOL and relf(M, ref["M"]) <= TOL and relf(X - x_in, ref["X"] - x_in) <= 2 * TOL, t
