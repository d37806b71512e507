"""The rule that gives a step's bf16 prompts to the kernel of 64 or of 128 positions per
workgroup (host code), at sizes where the wrong one measured 1.05 to 1.4 times the time."""
import pytest

from tests import gemm_plan as G


@pytest.mark.parametrize("heads,D,lens,long", [
    (2, 128, [8192], False), (8, 128, [4096], False), (4, 128, [6000, 6000], False), (12, 128, [4096], False),
    (16, 128, [2048, 2048], False), (32, 128, [300] * 16, False), (32, 128, [2048], True), (10, 128, [6000], True),
    (64, 128, [4096], True), (8, 128, [3000] * 3, True), (24, 128, [2048, 2048], True), (64, 128, [512] * 8, True),
    (4, 64, [8192], False), (6, 64, [6000, 6000], False), (10, 64, [3000] * 3, False), (8, 64, [6000], False),
    (32, 64, [2048], False), (32, 64, [1024] * 4, False), (32, 64, [4096], True), (16, 64, [8192], True),
    (16, 64, [6000, 6000], True), (10, 64, [8192] + [100] * 4, True)])
def test_prefill_kernel(heads, D, lens, long):
    assert G.prefill_long(heads, D, lens) == long
