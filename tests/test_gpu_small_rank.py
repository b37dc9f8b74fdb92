"""Ranks up to 192, whose factorisation and inverse one workgroup forms in one launch: edges of its 64 x 64 tiles, few and
many partial Gram matrices, a second pass that is cut short and one that is not, batches, and a breakdown in one of them."""
import numpy as np
import pytest

from paper_2504_05295_amd import inputs
from gpu_harness import GpuProblem, one_step_report

pytestmark = pytest.mark.gpu
MU, ETA = inputs.MU, inputs.ETA


@pytest.mark.parametrize("r", [1, 2, 63, 64, 65, 127, 128, 129, 191, 192])
@pytest.mark.parametrize("rows", [256, 2100])
@pytest.mark.parametrize("cond", [3.0, 1e3])
def test_conditioned_product(r, rows, cond):
    # B Q has singular values from 1 down to 1 / cond and no structure besides.  At 1e3 the first pass in fp32 leaves
    # ||P1^T P1 - I|| of up to cond^2 u = 6e-2, above the 1e-3 that cuts the second pass short.
    m, n = rows, 320
    rng = np.random.default_rng(7 * r + rows)
    a = np.linalg.qr(rng.standard_normal((m, r)))[0]
    v = np.linalg.qr(rng.standard_normal((n, r)))[0]
    o = np.linalg.qr(rng.standard_normal((r, r)))[0]
    g = ((a * np.logspace(0, -np.log10(cond), r)) @ v.T).astype(np.float32)
    gp = GpuProblem([(m, n, r)], False, "f32", q_raw=[np.ascontiguousarray(v @ o, dtype=np.float32)])
    gp.upload_grads([g])
    x_in, m_in, q_in = gp.host()
    assert gp.step(MU, ETA) == (0, -1)
    P1 = gp.debug(0, gp.B.DEBUG_P1)[:, :r].astype(np.float64)
    defect = np.linalg.norm(P1.T @ P1 - np.eye(r))
    # which way the second pass went: its factor, if it made one, is near the identity; the first pass' has the singular
    # values of B Q on its diagonal (one column: 1 in either, and nothing to be conditioned)
    factored = bool(np.abs(np.diag(gp.debug(0, gp.B.DEBUG_L))[:r] - 1).max() < 0.1)
    if r > 1:
        assert factored == (defect > 1e-3), (factored, defect)
    if cond < 10 or r == 1:
        assert defect < 1e-3, defect
    elif r >= 63:
        assert defect > 1e-3, defect
    rep, _ = one_step_report(gp, 0, x_in, m_in, q_in, g, MU, ETA, "lapack")
    # the forward error of a QR factor in fp32 is a few cond(B Q) u (6e-8), 1e-3 leaves the margin for r of them
    assert rep["X"] < 1e-4 and rep["M"] < 1e-4 and rep["orth"] < 1e-5, rep
    assert rep["dX"] < 1e-3 and rep["dM"] < 1e-3, rep


@pytest.mark.parametrize("math", ["f32", "bf16"])
def test_batch_with_a_breakdown(math):
    # (512, 256, 128) takes the split-bf16 products in bf16 mode; duplicate columns of Q make the middle B Q singular
    shapes = [(512, 256, 128)] * 3 + [(300, 200, 100)] * 2
    q_raw = [inputs.right_factor_raw(n, r, 5, i) for i, (m, n, r) in enumerate(shapes)]
    q_raw[1][:, 70] = q_raw[1][:, 3]
    gp = GpuProblem(shapes, True, math, q_raw=q_raw)
    grads = gp.grads_np(0)
    gp.upload_grads(grads)
    before = [gp.host(i) for i in range(len(shapes))]
    assert gp.step(MU, ETA) == (gp.B.DION_NUM_BREAKDOWN, 1)
    tol = 1e-4 if math == "f32" else 2e-2
    for i in range(len(shapes)):
        if i == 1:
            for u, w in zip(gp.host(i), before[i]):
                assert np.array_equal(u, w)
            continue
        rep, _ = one_step_report(gp, i, *before[i], gp.grad_as_f32(grads[i], True), MU, ETA, "lapack")
        assert rep["X"] <= tol and rep["M"] <= tol and rep["dX"] <= 2 * tol and rep["dM"] <= 2 * tol, (i, rep)


@pytest.mark.parametrize("lazy", [False, True])
def test_groups_side_by_side(lazy):
    # six shape groups of one matrix each, two of them on the split-bf16 path, on the caller's stream and the state's own: every step must give what the
    # matrices give in states of their own, bit for bit (the same kernels on the same data), also from a stream other than
    # the default one, captured into a graph that is replayed between eager work
    import torch
    shapes = [(512, 256, 128), (300, 200, 100), (256, 700, 64), (384, 512, 128), (256, 768, 128), (130, 1030, 40)]
    q_raw = [inputs.right_factor_raw(n, r, 5, i) for i, (m, n, r) in enumerate(shapes)]
    batch = GpuProblem(shapes, True, "bf16", q_raw=q_raw)
    single = [GpuProblem([s], True, "bf16", q_raw=[q_raw[i]], x0=[batch.x0[i]]) for i, s in enumerate(shapes)]
    side = torch.cuda.Stream()
    B = batch.B

    def compare():
        for i, p in enumerate(single):
            for u, w in zip(batch.host(i), p.host()):
                assert np.array_equal(u, w), (lazy, shapes[i])

    def step(p):
        return p.lazy_step(MU, ETA, True) if lazy else p.step(MU, ETA)

    grads = [batch.grads_np(t) for t in range(4)]
    batch.upload_grads(grads[0])
    for t in range(2):
        for i, g in enumerate(grads[t]):
            batch.G[i].copy_(torch.from_numpy(g.view(np.int16)).view(torch.bfloat16))
            single[i].upload_grads([g])
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            assert step(batch) == (0, -1)
        for p in single:
            assert step(p) == (0, -1)
        compare()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        if lazy:
            B.dion_lazy_step_batched(batch.state, batch.X, batch.G, batch.M, batch.Q, MU, ETA, True)
        else:
            B.dion_step_batched(batch.state, batch.X, batch.G, batch.M, batch.Q, MU, ETA)
    for t in range(2, 4):
        for i, g in enumerate(grads[t]):
            batch.G[i].copy_(torch.from_numpy(g.view(np.int16)).view(torch.bfloat16))
            single[i].upload_grads([g])
        graph.replay()
        torch.cuda.synchronize()
        assert B.dion_last_status(batch.state) == (0, -1)
        for p in single:
            assert step(p) == (0, -1)
        compare()
