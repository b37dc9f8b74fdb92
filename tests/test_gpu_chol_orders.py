"""The single-launch Cholesky factorisation at the sizes where its helpers deal out their tasks in another way (csrc/chol_panel.hip,
near_order): more panels than a round of the grid's rows, more near-diagonal tasks than workgroups, and beyond 64 panels, where
the inverse is a launch of its own; the rank-tolerant one there too."""
import pytest
import torch

from paper_2504_05295_amd import binding as B
from paper_2504_05295_amd import inputs

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA
U = 6e-8


def gaussian(seed, *shape):
    return torch.randn(shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


# (count, r): 36, 41, 48 and 59 panels on 15 x 17 behind the rows beyond the round, 62 from the front; 20 on 7 x 9 behind them, 25 and
# 31 at the far end; 65 and 91 panels without the inverse
@pytest.mark.parametrize("count,r", [(1, 2304), (1, 2600), (1, 3072), (1, 3750), (1, 3968), (2, 1280), (3, 1600), (2, 1984), (1, 4100), (1, 5800)])
def test_factor(count, r):
    # Z = G Q is the first r columns of a Gaussian m x n matrix, m = 2 r: condition about 5.8
    m, n, cond = 2 * r, r + 24, 6.0
    X = [torch.zeros((m, n), device="cuda") for _ in range(count)]
    M = [torch.empty((m, n), device="cuda") for _ in range(count)]
    Q = [torch.eye(n, r, device="cuda") for _ in range(count)]
    G = [gaussian(10 * r + i, m, n) for i in range(count)]
    st = B.dion_init_state([(m, n, r)] * count, B.DION_G_F32, B.DION_MATH_F32, M, Q)
    if count == 1:
        B.dion_step(st, X[0], G[0], M[0], Q[0], MU, ETA)
    else:
        B.dion_step_batched(st, X, G, M, Q, MU, ETA)
    assert B.dion_last_status(st) == (0, -1)
    for i in range(count):
        Z = B.dion_debug_buffer(st, i, B.DEBUG_Z)[:, :r].double()
        P1 = B.dion_debug_buffer(st, i, B.DEBUG_P1)[:, :r].double()
        L = torch.tril(B.dion_debug_buffer(st, i, B.DEBUG_L)[:r, :r].double())
        T = torch.linalg.cholesky(Z.T @ Z)
        # (the second pass is cut short; the Gram matrix carries U ||Z||^2, which the factor sees magnified by cond(Z), P1 by its square)
        u = U * r ** 0.5
        assert torch.linalg.norm(L - T) <= 8 * cond * u * torch.linalg.norm(T), (count, r, i)
        assert torch.linalg.norm(P1.T @ P1 - torch.eye(r, device="cuda", dtype=torch.float64)) <= 8 * cond ** 2 * u * r ** 0.5, (count, r, i)
        assert torch.linalg.norm(P1 @ T.T - Z) <= 8 * cond * u * torch.linalg.norm(Z), (count, r, i)


def test_rank_tolerant_factor_without_the_inverse():
    r1, r2, n = 64, 4100, 4160
    m = 2 * r2
    X, M1, M2, D = ([torch.zeros((m, n), device="cuda")] for _ in range(4))
    V1 = [gaussian(1, n, r1)]
    V2 = [torch.eye(n, r2, device="cuda")]
    dependent = [9, 700, 4099]
    for j in dependent:
        V2[0][:, j] = V2[0][:, j // 2]
    s1 = B.dion_init_state([(m, n, r1)], B.DION_G_F32, B.DION_MATH_F32, M1, V1)
    s2 = B.dion_init_state([(m, n, r2)], B.DION_G_F32, B.DION_MATH_F32, M2, V2)
    M2[0].copy_(gaussian(2, m, n))
    B.dion_double_step(s1, s2, X, [gaussian(3, m, n)], M1, V1, M2, V2, D, MU, MU, ETA)
    assert B.dion_last_status(s1) == (0, -1) and B.dion_last_status(s2) == (0, -1)
    null = B.dion_debug_buffer(s2, 0, B.DEBUG_NULL).reshape(-1)[:r2] != 0
    assert null.nonzero().reshape(-1).tolist() == dependent
    P = B.dion_debug_buffer(s2, 0, B.DEBUG_P)[:, :r2].double()
    assert (P.T @ P - torch.diag((~null).double())).abs().max() <= 1e-5     # the bound of the other fp32 tests
    R = B.dion_debug_buffer(s2, 0, B.DEBUG_R)[:, :r2].double()
    # M2 <- B - (1 - mu) P R^T, R = B^T P, and P spans B V2: B itself is what both give back
    Bm = M2[0].double() + (1 - MU) * (P @ R.T)
    Z = Bm[:, :r2]
    Z = Z[:, ~null]
    assert torch.linalg.norm(Z - P @ (P.T @ Z)) <= 1e-5 * torch.linalg.norm(Z)
    assert torch.linalg.norm(R - Bm.T @ P) <= 1e-5 * torch.linalg.norm(R)
