"""GPU parity of the duration-dependent path with up to eight labels on both sides of the size (K = 160) from which the backward scan
fetches table entries behind a block's last ones: one to four and more groups of sixteen durations a label."""
import numpy as np
import pytest

from paper_2604_18780_amd import synth
from test_gpu_durtrans import check, trans3_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,C", [(1, 8), (13, 2), (29, 8), (61, 7), (77, 1), (145, 8), (160, 8), (161, 8), (160, 3), (161, 3), (176, 8)])
def test_backward_scan_on_both_sides_of_its_choice(K, C):
    w = synth.small_random(10 * K + C, 3, 2 * K + 90, K, C, ragged=True)
    w.lengths[0] = w.T
    check(w, trans3_of(w, K), grad_logz=np.array([1.0, -0.5, 0.25]))
