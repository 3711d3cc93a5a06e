"""GPU parity of the duration-dependent path at the edges of its tiles: sixteen durations per matrix-core tile (one to four of
them), 64 durations per wave of the marginals (up to four groups), eight and sixteen labels per tile, and the sizes whose
windows do not fit the matrix-core kernels."""
import numpy as np
import pytest

from paper_2604_18780_amd import synth
from test_gpu_durtrans import check, trans3_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [3, 8, 9, 16, 17, 24, 32])
@pytest.mark.parametrize("K", [3, 4, 5, 15, 16, 17, 32, 33, 47, 48, 49, 63, 64])
def test_duration_tiles(K, C):
    w = synth.small_random(100 * K + C, 2, 150 + K, K, C, ragged=True)
    w.lengths[0] = w.T
    check(w, trans3_of(w, K), grad_logz=np.array([1.0, -0.5]))


@pytest.mark.parametrize("K,C", [(65, 8), (96, 20), (127, 8), (128, 16), (129, 8), (192, 5), (193, 8), (256, 16), (250, 3), (400, 8),
                                 (496, 8), (504, 8), (512, 8)])
def test_several_groups_of_durations(K, C):
    w = synth.small_random(K + C, 2, 2 * K + 37, K, C, ragged=False)
    w.lengths[:] = [w.T, K + 5]
    check(w, trans3_of(w, K))


@pytest.mark.parametrize("seed", [0, 1, 2, 3, 4, 5, 1073057435])
@pytest.mark.parametrize("K,C,delta", [(5, 17, 64), (4, 6, 40), (12, 20, 48), (400, 8, 0)])
def test_backward_scans_whose_forward_rows_were_scanned_again(seed, K, C, delta):
    """The backward scan weights what starts and ends at a position with the forward rows.  Weak emissions and banded transitions
    are forgotten so slowly that one direction can be verified at an attempt at which the other is not."""
    w = synth.small_random(seed, 3, 113 if delta else 1500, K, C, ragged=True, scale=0.05)
    w.lengths[0] = w.T
    w.trans[:] = synth.reshape_transitions(w.trans, sd=0.1, band=2)
    check(w, trans3_of(w, seed % 1000), ckpt_interval=delta)
