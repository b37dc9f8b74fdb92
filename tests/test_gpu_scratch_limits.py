"""Workspaces without room for the padded copies of the ragged update (the update then runs on the general core), and the static
workspace where it holds what a call of another shape left there."""
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, relf

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA


def up(x, k):
    return (x + k - 1) // k * k


def test_state_without_room_for_the_copies():
    import torch
    from paper_2504_05295_amd import binding as B
    m, n, r = 5003, 2999, 360
    gp = GpuProblem([(m, n, r)], True, "bf16", seed=11)
    need = B.dion_workspace_bytes([(m, n, r)], B.DION_G_BF16, B.DION_MATH_BF16)
    copies = 2 * up(r, 64) * (up(m, 256) + 2 * up(n, 128))
    X, M, Q = gp.X[0].clone(), torch.empty_like(gp.M[0]), torch.from_numpy(gp.q_raw[0].copy()).cuda()
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    off = -ws.data_ptr() % 256
    with pytest.raises(B.DionError) as e:
        B.dion_init_state([(m, n, r)], B.DION_G_BF16, B.DION_MATH_BF16, [M], [Q], workspace=ws[off:off + need - copies - 1])
    assert e.value.code == B.DION_EWORKSPACE
    ws[off + need - copies:] = 0x5a
    st = B.dion_init_state([(m, n, r)], B.DION_G_BF16, B.DION_MATH_BF16, [M], [Q], workspace=ws[off:off + need - copies])
    for t in range(2):
        gp.upload_grads(gp.grads_np(t))
        assert gp.step(MU, ETA) == (0, -1)
        B.dion_step(st, X, gp.G[0], M, Q, MU, ETA)
        torch.cuda.synchronize()
        # the same bf16 factors, 360 products of which are summed in fp32 in another order; a difference of 1e-6 in M may move a
        # bf16 operand of the next step by one place, 2^-9, in few of its elements
        tol = 1e-5 if t == 0 else 2e-3
        for u, v in ((X, gp.X[0]), (M, gp.M[0]), (Q, gp.Q[0])):
            assert relf(u.cpu().numpy(), v.cpu().numpy()) <= tol, t
    assert bool((ws[off + need - copies:] == 0x5a).all())


@pytest.mark.parametrize("before", [(1500, 1500, 200), (700, 2000, 300)])
def test_static_after_another_shape(before):
    import torch
    from paper_2504_05295_amd import binding as B
    for shape, math in ((before, "f32"), ((1024, 1024, 256), "bf16"), ((512, 1024, 256), "bf16")):
        code = B.DION_MATH_BF16 if math == "bf16" else B.DION_MATH_F32
        ref = GpuProblem([shape], True, math, seed=13)
        X, M, Q = ref.X[0].clone(), ref.M[0].clone(), ref.Q[0].clone()
        ref.upload_grads(ref.grads_np(0))
        assert ref.step(MU, ETA) == (0, -1)
        B.dion_step_static(X, ref.G[0], M, Q, B.DION_G_BF16, code, MU, ETA)
        torch.cuda.synchronize()
        for u, v in ((X, ref.X[0]), (M, ref.M[0]), (Q, ref.Q[0])):
            if math == "bf16":
                assert torch.equal(u, v), shape
            else:   # (the static workspace may hold a plan without splits: sums in another order)
                assert relf(u.cpu().numpy(), v.cpu().numpy()) <= 1e-5, shape
