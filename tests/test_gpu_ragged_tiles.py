"""Parity where the tiles of the general GEMM core meet the edges of their matrices: dimensions one below, at and one above
a tile (64, 128) and a slab of the contraction (32, 64), and outputs narrower than a tile next to long contractions."""
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, one_step_report

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA


@pytest.mark.parametrize("shape", [(64, 64, 32), (65, 66, 31), (63, 200, 33), (127, 129, 63), (128, 130, 64), (129, 191, 65),
                                   (70, 3000, 61), (3000, 70, 64), (1030, 1157, 97), (2050, 1090, 129), (1153, 2177, 33)])
@pytest.mark.parametrize("g_bf16,math", [(False, "f32"), (True, "f32"), (False, "bf16"), (True, "bf16")])
def test_edges_of_tiles(shape, g_bf16, math):
    tol = 1e-4 if math == "f32" else 2e-2    # the bounds of the fixed-shape parity tests
    gp = GpuProblem([shape], g_bf16, math, seed=3)
    for t in range(2):
        g = gp.grads_np(t)[0]
        x_in, m_in, q_in = gp.host()
        gp.upload_grads([g])
        assert gp.step(MU, ETA) == (0, -1), (shape, t)
        rep, _ = one_step_report(gp, 0, x_in, m_in, q_in, gp.grad_as_f32(g, g_bf16), MU, ETA, "lapack")
        assert rep["X"] <= tol and rep["M"] <= tol and rep["dX"] <= 2 * tol and rep["dM"] <= 2 * tol, (shape, t, rep)
        assert rep["orth"] <= (1e-5 if math == "f32" else 1e-3), (shape, t, rep)


@pytest.mark.parametrize("lazy", [False, True])
def test_more_blocks_of_rows_than_a_second_grid_axis_takes(lazy):
    # 65625 blocks of 32 rows when the factor's columns are scaled; 65536 is the end of a grid's second axis
    from oracle import dion_oracle as orc
    from gpu_harness import relf
    shape = (9, 2100000, 4)
    gp = GpuProblem([shape], True, "f32")
    g = gp.grads_np(0)[0]
    x_in, m_in, q_in = gp.host()
    gp.upload_grads([g])
    g32 = gp.grad_as_f32(g, True)
    if lazy:
        assert gp.lazy_step(MU, ETA, True) == (0, -1)
        ref = orc.lazy_dion_step(x_in, g32, m_in, q_in, MU, ETA, True, "lapack")
        q_ref = ref["V"]
    else:
        assert gp.step(MU, ETA) == (0, -1)
        ref = orc.dion_step(x_in, g32, m_in, q_in, MU, ETA, "lapack")
        q_ref = ref["Q"]
    X, M, Q = gp.host()
    # (the update itself, eta sqrt(m / n) / sqrt(n) an entry, is what X's last bit resolves here: the factor is compared instead)
    assert relf(X, ref["X"]) <= 1e-4 and relf(M, ref["M"]) <= 1e-4 and relf(Q, q_ref) <= 1e-4
