"""Which forward-only calls halve the automatic interval: the plan's rule, read off the workspace it asks for (an explicit
interval is never halved, so the sizes differ exactly where the rule halves)."""
import pytest

from paper_2604_18780_amd import binding as sb


@pytest.mark.parametrize("B,T,K,C,halved", [
    (4, 100_000, 64, 24, True),     # interval 392, warm-up 96
    (4, 102_400, 64, 24, True),     # 400
    (4, 73_728, 64, 24, False),     # 288: a task would spend half its time on its warm-up
    (4, 49_152, 64, 24, False),     # 192
    (4, 40_960, 64, 24, False),     # 160
    (4, 32_768, 16, 24, True),      # 128, warm-up 32
    (4, 24_576, 16, 24, False),     # 96
    (4, 16_384, 16, 24, False),     # 64
    (4, 49_152, 32, 64, False),     # one task per SIMD is all there is room for
    (1, 400_000, 512, 8, False),
])
def test_halved_from_four_warm_ups_on(B, T, K, C, halved):
    auto = sb.semicrf_ckpt_interval(B, T, K, C)
    same = sb.semicrf_workspace_bytes(B, T, K, C, 0, 0) == sb.semicrf_workspace_bytes(B, T, K, C, auto, 0)
    assert same == (not halved), auto
