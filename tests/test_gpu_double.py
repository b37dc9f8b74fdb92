"""GPU parity of the Double Dion step (Section 5.2) through the C-ABI against the CPU oracle, step by step from
the GPU's own state; fp32 and bf16 operand modes, single and batched, and the two breakdown cases."""
import numpy as np
import pytest
import torch

from oracle import dion_oracle as orc
from paper_2504_05295_amd import inputs, binding as B
from gpu_harness import relf

pytestmark = pytest.mark.gpu
MU1, MU2, ETA = 0.999, 0.95, inputs.ETA          # the paper's beta1 = 0.001, beta2 = 0.05


class DoubleProblem:
    def __init__(self, shapes, r1, r2, g_bf16, math, v1_raw=None, v2_raw=None, warm=True):
        self.shapes, self.r1, self.r2, self.g_bf16 = shapes, r1, r2, g_bf16
        dev = "cuda"
        cnt = len(shapes)
        self.X = [torch.from_numpy(inputs.weight(m, n, 1, i)).to(dev) for i, (m, n) in enumerate(shapes)]
        self.M1 = [torch.empty((m, n), dtype=torch.float32, device=dev) for (m, n) in shapes]
        self.M2 = [torch.empty((m, n), dtype=torch.float32, device=dev) for (m, n) in shapes]
        self.D = [torch.empty((m, n), dtype=torch.float32, device=dev) for (m, n) in shapes]
        v1 = v1_raw or [inputs.right_factor_raw(n, r1, 2, i) for i, (m, n) in enumerate(shapes)]
        v2 = v2_raw or [inputs.right_factor_raw(n, r2, 3, i) for i, (m, n) in enumerate(shapes)]
        self.V1 = [torch.from_numpy(v.copy()).to(dev) for v in v1]
        self.V2 = [torch.from_numpy(v.copy()).to(dev) for v in v2]
        mth = B.DION_MATH_BF16 if math == "bf16" else B.DION_MATH_F32
        self.s1 = B.dion_init_state([(m, n, r1) for (m, n) in shapes], B.DION_G_BF16 if g_bf16 else B.DION_G_F32, mth,
                                    self.M1, self.V1)
        self.s2 = B.dion_init_state([(m, n, r2) for (m, n) in shapes], B.DION_G_F32, mth, self.M2, self.V2)
        if warm:
            # as after many steps: M2 has full rank (from M2 = 0 it is a sum of rank-r1 sketches, see the cold-start test)
            for i, (m, n) in enumerate(shapes):
                self.M2[i].copy_(torch.from_numpy(inputs.gaussian((m, n), 3e-2, 7, 11, 0, i)))
        self.G = [None] * cnt

    def upload(self, grads):
        for i, g in enumerate(grads):
            t = torch.from_numpy(g.view(np.int16)).view(torch.bfloat16) if self.g_bf16 else torch.from_numpy(g)
            self.G[i] = t.to("cuda")

    def step(self):
        B.dion_double_step(self.s1, self.s2, self.X, self.G, self.M1, self.V1, self.M2, self.V2, self.D, MU1, MU2, ETA)
        return B.dion_last_status(self.s1), B.dion_last_status(self.s2)

    def host(self, i):
        return [t[i].cpu().numpy() for t in (self.X, self.M1, self.V1, self.M2, self.V2)]


def oracle_with_gpu_decisions(dp, i, x, g32, m1, v1, m2, v2, method, band=2.0):
    """The oracle step of matrix i with the dependent / independent decisions of stage 2 taken as the library took them
    in its own precision (both sides have to take a decision that floating point makes in the same precision), after
    checking that every one of them is right or borderline: with the squared relative distances r_j that the oracle
    finds along that sequence of decisions, kept columns have r_j > RANK_TOL / band, dropped ones r_j < RANK_TOL * band."""
    r2 = v2.shape[1]
    null = B.dion_debug_buffer(dp.s2, i, B.DEBUG_NULL).cpu().numpy().reshape(-1)[:r2]
    gpu_keep = null == 0
    ref = orc.double_dion_step(x, g32, m1, v1, m2, v2, MU1, MU2, ETA, method, forced=gpu_keep.astype(int))
    r = ref["ratio"]
    assert np.all(r[gpu_keep] > orc.RANK_TOL / band), ("kept a dependent column", np.sort(r[gpu_keep])[:4])
    assert np.all(r[~gpu_keep] < orc.RANK_TOL * band), ("dropped an independent column", np.sort(r[~gpu_keep])[-4:])
    return ref


def run(shapes, r1, r2, g_bf16, math, steps, tol, method="householder", warm=True, dx_tol=None):
    dp = DoubleProblem(shapes, r1, r2, g_bf16, math, warm=warm)
    for t in range(steps):
        grads = [inputs.gradient(m, n, t, 0, i, bf16=g_bf16) for i, (m, n) in enumerate(shapes)]
        before = [dp.host(i) for i in range(len(shapes))]
        dp.upload(grads)
        assert dp.step() == ((0, -1), (0, -1))
        for i in range(len(shapes)):
            g32 = inputs.bf16_bits_to_f32(grads[i]) if g_bf16 else grads[i]
            x, m1, v1, m2, v2 = before[i]
            ref = oracle_with_gpu_decisions(dp, i, x, g32, m1, v1, m2, v2, method)
            X, M1, V1, M2, V2 = dp.host(i)
            kept = int(ref["keep"].sum())
            assert np.array_equal(V2[:, ~ref["keep"]], v2[:, ~ref["keep"]])       # dependent columns keep their factor
            assert abs(np.linalg.norm(X.astype(np.float64) - x) / (ETA * np.sqrt(shapes[i][0] / shapes[i][1]) * np.sqrt(kept)) - 1) < 10 * tol
            err = dict(X=relf(X, ref["X"]), M1=relf(M1, ref["M1"]), M2=relf(M2, ref["M2"]),
                       dX=relf(X.astype(np.float64) - x, ref["X"] - x), D=relf(dp.D[i].cpu().numpy(), ref["D"]),
                       v1=float(np.min(np.abs(np.sum(V1.astype(np.float64) * ref["V1"], axis=0)))),
                       v2=float(np.min(np.abs(np.sum(V2.astype(np.float64) * ref["V2"], axis=0)))))
            assert max(err["X"], err["M1"], err["M2"], err["D"]) <= tol and err["dX"] <= 3 * tol, (t, i, err)
            print("double step", t, shapes[i], (r1, r2), "independent columns in stage 2:", kept, {k: "%.2e" % v for k, v in err.items()}, flush=True)
            assert max(err["X"], err["M1"], err["M2"], err["D"]) <= tol and err["dX"] <= (dx_tol or 3 * tol), (t, i, err)
            assert err["v1"] > 1 - 10 * tol and (err["v2"] > 1 - 10 * tol or dx_tol), (t, i, err)


def test_double_dion_fp32():
    run([(256, 192)], 8, 32, False, "f32", 3, 1e-4)
    run([(200, 136), (200, 136), (128, 384)], 8, 24, False, "f32", 2, 1e-4)


def test_double_dion_bf16_large_tile_path():
    run([(512, 256), (256, 768)], 128, 128, True, "bf16", 2, 2e-2)


def test_double_dion_bf16_full_size_direct_load_path():
    # 8192 x 8192 with r2 = 1024: stage 2 reads the stored bf16 copies of M2 + sketch.  Once from a full-rank M2 and once
    # from M2 = 0, where the buffer of stage 2 has rank r1 = 256 and three quarters of its columns are dependent.
    run([(8192, 8192)], 256, 1024, True, "bf16", 1, 2e-2, method="lapack")
    # (while the buffer fills up the independent columns are badly conditioned among themselves, so the bf16 rounding of
    # the operands, 3e-3 per entry of B2 V2, weighs more on the update's direction than in a full-rank step)
    run([(8192, 8192)], 256, 1024, True, "bf16", 2, 2e-2, method="lapack", warm=False, dx_tol=0.15)


def test_double_dion_stage_one_breakdown_and_dependent_column_in_stage_two():
    m, n, r1, r2 = 256, 192, 8, 32
    good1 = [inputs.right_factor_raw(n, r1, 2, i) for i in range(2)]
    good2 = [inputs.right_factor_raw(n, r2, 3, i) for i in range(2)]
    bad1 = good1[1].copy(); bad1[:, 5] = bad1[:, 2]
    bad2 = good2[1].copy(); bad2[:, 9] = bad2[:, 4]
    grads = [inputs.gradient(m, n, 0, 0, i, bf16=False) for i in range(2)]
    # stage 1 of matrix 1 fails: that matrix is left alone entirely, its neighbour is stepped
    dp = DoubleProblem([(m, n)] * 2, r1, r2, False, "f32", v1_raw=[good1[0], bad1])
    before = [dp.host(i) for i in range(2)]
    dp.upload(grads)
    st1, st2 = dp.step()
    assert st1 == (B.DION_NUM_BREAKDOWN, 1) and st2 == (B.DION_NUM_BREAKDOWN, 1)
    for u, v in zip(before[1], dp.host(1)):
        assert np.array_equal(u, v)
    ref = orc.double_dion_step(*before[0][:1], grads[0], *before[0][1:], MU1, MU2, ETA)
    assert relf(dp.host(0)[0], ref["X"]) < 1e-4
    # V2 of matrix 1 has two identical columns: no failure, the second of them is dependent, takes no part in the step
    # and stays as it was; everything else is the step on the other 31 columns
    dp = DoubleProblem([(m, n)] * 2, r1, r2, False, "f32", v2_raw=[good2[0], bad2])
    before = [dp.host(i) for i in range(2)]
    dp.upload(grads)
    assert dp.step() == ((0, -1), (0, -1))
    X, M1, V1, M2, V2 = dp.host(1)
    ref = oracle_with_gpu_decisions(dp, 1, before[1][0], grads[1], before[1][1], before[1][2], before[1][3], before[1][4], "householder")
    assert ref["status"] == orc.STATUS_OK and int(ref["keep"].sum()) == r2 - 1 and not ref["keep"][9]
    assert np.array_equal(V2[:, 9], before[1][4][:, 9])
    assert relf(X, ref["X"]) < 1e-4 and relf(M2, ref["M2"]) < 1e-4 and relf(M1, ref["M1"]) < 1e-4
    assert relf(X.astype(np.float64) - before[1][0], ref["X"] - before[1][0]) < 3e-4
    assert float(np.min(np.abs(np.sum(V2.astype(np.float64) * ref["V2"], axis=0)))) > 1 - 1e-3


@pytest.mark.parametrize("r2,links", [(192, 128), (512, 256)])       # a launch per panel, and all panels in one launch
def test_column_dropped_in_the_second_pass_stays_dropped_in_the_last(r2, links):
    # B2 V2 built column by column: V2 is the first columns of the identity, M2 holds the columns, stage 1 adds nothing to
    # speak of.  Chains z_0 = q_0, z_l = c q_(l-1) + s q_l with s^2 > RANK_TOL have condition (c / s)^l: in fp32 the pivots
    # of the first pass are rounding noise from the fourth link on.  Behind them, in later panels, a column that lies
    # in the span of each chain: where the noise was positive the first pass takes it for a column of its own, the second
    # finds it dependent.  A few longer chains leave the second pass' result away from orthonormal, so that the last
    # pass is not cut short and has to drop those columns again.  (What the noise does differs from seed to seed: seeds that
    # do not get there, or whose second pass leaves more than the last one's pivot bounds allow, say nothing here.)
    m, n, r1 = 1024, 512, 8
    chains = [(4, 0.04)] * ((links - 36) // 4) + [(6, 0.06)] * 6
    checked = 0
    for seed in range(10):
        q = np.linalg.qr(np.random.default_rng(seed).standard_normal((m, r2)))[0]
        coef = np.eye(r2)
        pos = 0
        for k, (length, s) in enumerate(chains):
            for l in range(1, length):
                coef[:, pos + l] = 0.0
                coef[pos + l - 1, pos + l], coef[pos + l, pos + l] = np.sqrt(1.0 - s * s), s
            coef[:, links + k] = 0.0
            coef[pos + length - 1, links + k] = 1.0
            pos += length
        z = (q @ coef).astype(np.float32)
        dp = DoubleProblem([(m, n)], r1, r2, False, "f32", v2_raw=[np.eye(n, r2, dtype=np.float32)], warm=False)
        dp.M2[0][:, :r2].copy_(torch.from_numpy(z))
        dp.upload([inputs.gaussian((m, n), 1e-9, 3, 1, 0, 0)])
        st1, st2 = dp.step()
        debug = lambda which: B.dion_debug_buffer(dp.s2, 0, which).cpu().numpy().astype(np.float64)
        p1, p2, p = (debug(w)[:, :r2] for w in (B.DEBUG_P1, B.DEBUG_Z, B.DEBUG_P))     # of the three passes
        keep1, keep2 = (np.abs(x).max(axis=0) > 0 for x in (p1, p2))
        ev = np.linalg.eigvalsh(p2[:, keep2].T @ p2[:, keep2])
        defect = np.linalg.norm(p2.T @ p2 - np.diag(keep2.astype(float)))
        print("r2", r2, "seed", seed, "dropped in the first pass", int(np.sum(~keep1)), "in the second", int(np.sum(keep1 & ~keep2)),
              "defect after it %.2e" % defect, "eigenvalues %.2e to %.2e" % (ev[0], ev[-1]), st2, flush=True)
        if not (np.any(keep1 & ~keep2) and defect > 1e-3 and ev[0] > 0.1 and ev[-1] < 10):     # (pivots lie between these)
            continue
        checked += 1
        assert st1 == (0, -1) and st2 == (0, -1)
        null = debug(B.DEBUG_NULL).reshape(-1)[:r2] != 0
        assert np.all(null >= ~keep2)
        assert np.abs(p.T @ p - np.diag((~null).astype(float))).max() < 1e-5     # the bound of the other fp32 tests
    assert checked >= 3


def test_double_dion_cold_start_moves_the_weights_from_the_first_step():
    # from M2 = 0 the buffer of stage 2 has rank r1, 2 r1, ...: the step uses the rank that is there.  While the buffer
    # fills up, the independent columns of B2 V2 are badly conditioned among themselves (squared relative distances down
    # to RANK_TOL, condition numbers of a few thousand), which amplifies the forward error of any QR factor: the bound on
    # the update's error is wider on those steps, the one on X, M1, M2 is the usual one.
    for (m, n, r1, r2, g_bf16, math, tol, dx_tol) in [(256, 192, 16, 32, False, "f32", 1e-4, 3e-3), (1024, 768, 128, 512, True, "bf16", 2e-2, 0.15)]:
        dp = DoubleProblem([(m, n)], r1, r2, g_bf16, math, warm=False)
        ranks = []
        for t in range(5):
            g = inputs.gradient(m, n, t, 0, 0, bf16=g_bf16)
            g32 = inputs.bf16_bits_to_f32(g) if g_bf16 else g
            x, m1, v1, m2, v2 = dp.host(0)
            dp.upload([g])
            assert dp.step() == ((0, -1), (0, -1))
            ref = oracle_with_gpu_decisions(dp, 0, x, g32, m1, v1, m2, v2, "lapack")
            X, M1, V1, M2, V2 = dp.host(0)
            k = int(ref["keep"].sum())
            ranks.append(k)
            dx = np.linalg.norm(X.astype(np.float64) - x)
            edx = relf(X.astype(np.float64) - x, ref["X"] - x)
            print((m, n, r1, r2), "step", t, "independent columns", k, "X %.2e M2 %.2e dX %.2e" % (relf(X, ref["X"]), relf(M2, ref["M2"]), edx), flush=True)
            assert abs(dx / (ETA * np.sqrt(m / n) * np.sqrt(k)) - 1) < 10 * tol          # the weights move, by the rank that is there
            assert relf(X, ref["X"]) < tol and relf(M2, ref["M2"]) < tol and relf(M1, ref["M1"]) < tol, t
            assert edx < (3 * tol if t == 0 else dx_tol), (t, edx)
            assert np.array_equal(V2[:, ~ref["keep"]], v2[:, ~ref["keep"]])
            assert np.abs(np.linalg.norm(V2.astype(np.float64), axis=0) - 1).max() < 1e-5
        print("independent columns per step:", ranks, flush=True)
        assert r1 - 2 <= ranks[0] <= r1 and ranks[1] > ranks[0] and ranks[-1] > ranks[1]       # the rank grows as M2 fills up
