"""The update of matrices of any size on the direct-load core (bf16 operands, large matrices): sizes around
whole tiles, rows at every alignment, ranks around a slab of the contraction, both storage types of G, and nothing
written beside the matrices."""
import numpy as np
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, one_step_report, relf

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA
GUARD = 4096   # elements on either side (a multiple of 4: the matrices stay 16-byte aligned)


def guarded(t):
    import torch
    flat = torch.full((t.numel() + 2 * GUARD,), 12345.0, dtype=t.dtype, device=t.device)
    view = flat[GUARD:GUARD + t.numel()].view(t.shape)
    view.copy_(t)
    return flat, view


def guards_intact(flat):
    return bool((flat[:GUARD] == 12345.0).all()) and bool((flat[-GUARD:] == 12345.0).all())


# (400 tiles and r = 256 upwards, 352 with two or three last columns, or 1024 tiles and r = 72 upwards, two thirds of whole rounds of 256 tiles used; the last two are
# the general core's: a rank or a round short of that)
@pytest.mark.parametrize("shape", [(5003, 2999, 360), (2815, 5121, 256), (20001, 703, 353), (703, 20002, 352), (8191, 4097, 72), (5003, 2999, 351),
                                   (4097, 4095, 256)])
@pytest.mark.parametrize("g_bf16", [False, True])
def test_edges(shape, g_bf16):
    tol = 2e-2   # the bound of the fixed-shape parity tests in bf16 mode
    gp = GpuProblem([shape], g_bf16, "bf16", seed=5)
    fx, gp.X[0] = guarded(gp.X[0])
    fm, gp.M[0] = guarded(gp.M[0])
    for t in range(2):
        g = gp.grads_np(t)[0]
        x_in, m_in, q_in = gp.host()
        gp.upload_grads([g])
        assert gp.step(MU, ETA) == (0, -1), (shape, t)
        assert guards_intact(fx) and guards_intact(fm), (shape, t)
        rep, ref = one_step_report(gp, 0, x_in, m_in, q_in, gp.grad_as_f32(g, g_bf16), MU, ETA, "lapack")
        assert rep["X"] <= tol and rep["M"] <= tol and rep["dX"] <= 2 * tol and rep["dM"] <= 2 * tol, (shape, t, rep)
        # last rows and columns by themselves, where the last tiles are
        X, M, _ = gp.host()
        for a, b in ((X, ref["X"]), (M, ref["M"])):
            assert relf(a[-1], b[-1]) <= tol and relf(a[:, -1], b[:, -1]) <= tol, (shape, t)


def test_batch_and_lazy():
    shapes = [(5003, 2999, 360)] * 2 + [(1030, 1157, 33)]
    gp = GpuProblem(shapes, True, "bf16", seed=6)
    grads = gp.grads_np(0)
    gp.upload_grads(grads)
    before = [gp.host(i) for i in range(len(shapes))]
    assert gp.step(MU, ETA) == (0, -1)
    for i in range(len(shapes)):
        rep, _ = one_step_report(gp, i, *before[i], gp.grad_as_f32(grads[i], True), MU, ETA, "lapack")
        assert rep["X"] <= 2e-2 and rep["M"] <= 2e-2 and rep["dX"] <= 4e-2 and rep["dM"] <= 4e-2, (i, rep)
    from oracle import dion_oracle as orc
    gp = GpuProblem([(5003, 2999, 360)], True, "bf16", seed=7)
    g = gp.grads_np(0)[0]
    gp.upload_grads([g])
    x_in, m_in, q_in = gp.host()
    assert gp.lazy_step(MU, ETA, True) == (0, -1)
    ref = orc.lazy_dion_step(x_in, gp.grad_as_f32(g, True), m_in, q_in, MU, ETA, True, "lapack")
    X, M, _ = gp.host()
    assert relf(X - x_in, ref["X"] - x_in) <= 4e-2 and relf(M, ref["M"]) <= 2e-2
