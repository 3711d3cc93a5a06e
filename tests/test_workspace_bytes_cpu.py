"""What semicrf_fwd_bwd_static accepts, from the host-only semicrf_workspace_bytes (no GPU)."""
import pytest

from paper_2604_18780_amd import binding as sb


@pytest.mark.parametrize("B,T,K,C", [(64, 4054, 8, 8), (64, 2778, 64, 5)])
def test_the_choice_of_the_warm_up_takes_no_room_of_its_own(B, T, K, C):
    """The longest sequences of these shapes that the static array holds without that choice's arrays."""
    limit = sb.SEMICRF_STATIC_WORKSPACE_BYTES
    assert limit - 32768 < sb.semicrf_workspace_bytes(B, T, K, C, 0, 1) <= limit
