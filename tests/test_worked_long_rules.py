"""Worked expression with a long sum: the sizes whose contractions go to the bf16 matrix cores, which ask for more workspace than the family's kernels (no GPU)."""
import pytest

from paper_1711_01348_amd import binding as B
from paper_1711_01348_amd import workloads as wl


def families_bytes(I, J, K):
    up = lambda n: (n + 255) // 256 * 256
    return up(16 * I) + up(4 * J) + up(8 * (I + J) * K * 4) + up(8 * (2 * I + J) * 4)


@pytest.mark.parametrize("I,J,K,taken", [
    (1024, 1024, 64, True), (1024, 1020, 64, False), (64, 32768, 64, True),             # narrow tiles: whatever the shape
    (1400, 1400, 96, True), (1024, 1024, 96, False), (192, 30720, 128, True), (64, 32768, 96, False), (160, 32768, 128, False),
    (128, 16384, 192, True), (64, 32768, 192, False), (180, 11000, 224, True), (128, 16384, 256, False), (16384, 128, 512, False),
    (256, 16384, 512, True), (2048, 2048, 544, False), (160, 32000, 256, True), (128, 65536, 256, False)])   # (160 rows: the forward pass alone)
def test_sizes_on_the_bf16_matrix_cores(I, J, K, taken):
    plan = B.Plan(wl.worked_expr(I, J, K, "f32"))
    assert plan.forward_family == "worked_mfma"
    assert (plan.workspace_bytes > families_bytes(I, J, K)) == taken
    assert taken or plan.workspace_bytes == families_bytes(I, J, K)
