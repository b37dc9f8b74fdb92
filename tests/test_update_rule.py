"""Which matrices of bf16 mode off the large tiles take the direct-load update, seen on the CPU: the workspace then holds the
padded bf16 copies of the three factors, which fp32 mode never asks for."""
import pytest

from paper_2504_05295_amd import binding as B


def up(x, k):
    return (x + k - 1) // k * k


@pytest.mark.parametrize("m,n,r,direct", [
    (5003, 2999, 375, True), (5003, 2999, 352, True), (5003, 2999, 351, False), (5003, 3001, 256, True), (5003, 3001, 255, False),
    (2815, 5121, 256, True), (4097, 4095, 256, False), (2500, 2500, 1000, False),
    (8191, 4097, 72, True), (8191, 4097, 71, False), (16383, 2047, 80, False), (7300, 4608, 72, True),
    # rows on 16 bytes but not on whole lines: from r = 100 on
    (4526, 25616, 90, False), (4526, 25616, 99, False), (4526, 25616, 100, True), (4526, 25617, 90, True), (4621, 14000, 96, False),
])
def test_direct_update(m, n, r, direct):
    need = B.dion_workspace_bytes([(m, n, r)], B.DION_G_BF16, B.DION_MATH_BF16)
    plain = B.dion_workspace_bytes([(m, n, r)], B.DION_G_BF16, B.DION_MATH_F32)
    assert need - plain == (2 * up(r, 64) * (up(m, 256) + 2 * up(n, 128)) if direct else 0)
