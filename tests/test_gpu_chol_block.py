"""The 64 x 64 diagonal block of the Cholesky factorisation, formed in steps of 16 columns by three waves: edges of the steps
and of the block in each driver (one workgroup up to r = 192, single launch from there, launch per panel), through the factor
of the first Cholesky-QR pass that a step leaves in the workspace."""
import numpy as np
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA


@pytest.mark.parametrize("r", [1, 3, 15, 16, 17, 31, 33, 47, 48, 49, 64, 80, 113, 192, 193, 255, 272])
@pytest.mark.parametrize("cond", [2.0, 60.0])
def test_factor_and_inverse(r, cond):
    # B Q = A diag(s) O with orthonormal A and a rotation O: every pivot depends on all columns before it
    m, n = 640, 320
    rng = np.random.default_rng(r)
    a = np.linalg.qr(rng.standard_normal((m, r)))[0]
    v = np.linalg.qr(rng.standard_normal((n, r)))[0]
    o = np.linalg.qr(rng.standard_normal((r, r)))[0]
    g = ((a * np.logspace(0, -np.log10(cond), r)) @ v.T).astype(np.float32)
    gp = GpuProblem([(m, n, r)], False, "f32", q_raw=[np.ascontiguousarray(v @ o, dtype=np.float32)])
    gp.upload_grads([g])
    assert gp.step(MU, ETA) == (0, -1)
    Z = gp.debug(0, gp.B.DEBUG_Z)[:, :r].astype(np.float64)
    P1 = gp.debug(0, gp.B.DEBUG_P1)[:, :r].astype(np.float64)
    # (the second pass is cut short at these condition numbers; tiles above the block diagonal are nobody's)
    L = np.tril(gp.debug(0, gp.B.DEBUG_L)[:r, :r].astype(np.float64))
    T = np.linalg.qr(Z)[1]
    T *= np.sign(np.diag(T))[:, None]
    # u = 6e-8: the Gram matrix carries u ||Z||^2, which the factor sees magnified by cond(Z), P1 by its square
    u = 6e-8 * np.sqrt(r)
    assert np.linalg.norm(L - T.T) <= 8 * cond * u * np.linalg.norm(T), (r, cond)
    assert np.linalg.norm(P1.T @ P1 - np.eye(r)) <= 8 * cond ** 2 * u * np.sqrt(r), (r, cond)
    assert np.linalg.norm(P1 @ T - Z) <= 8 * cond * u * np.linalg.norm(Z), (r, cond)
