"""The Viterbi decode's rule for ties: smallest duration, then smallest label, among candidates whose scores differ by no more than
rounding.  A run of one label that is longer than K can be cut into the same durations in any order at the same score, so
such shapes are full of ties; which of two equal sums comes out larger in the last bit depends on the order of additions,
and so on how the scan was cut into intervals.  The path must not.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_viterbi import check, dev

pytestmark = pytest.mark.gpu


def runs(seed, B, T, K, C, length, level):
    """Runs of one label, about `length` tokens each, the label of a run `level` above the others, unit noise."""
    w = synth.small_random(seed, B, T, K, C, ragged=False)
    rng = np.random.default_rng(seed + 1)
    w.lengths[:] = rng.integers(T // 2, T + 1, size=B)
    w.lengths[0] = T
    for b in range(B):
        which = (rng.random(T) < 1.0 / length).cumsum()
        label = rng.integers(0, C, T + 1)[which]
        w.emis[b, np.arange(T), label] += level
    return w


def decode(w, flags):
    out = sb.semicrf_viterbi(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), flags=flags)
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("T,K,C,length,level", [
    (3000, 8, 4, 40, 2.0), (3000, 8, 4, 40, 12.0), (6000, 57, 3, 150, 2.0), (6000, 57, 3, 400, 8.0), (4000, 16, 8, 60, 3.0),
    (20000, 5, 3, 100, 30.0), (3000, 90, 5, 300, 4.0), (2000, 12, 24, 80, 6.0), (1500, 20, 64, 90, 8.0),
    (1200, 9, 15, 60, 4.0), (1200, 9, 16, 60, 4.0), (1200, 9, 17, 60, 4.0), (1200, 33, 32, 60, 4.0), (1200, 33, 33, 60, 4.0),
    (3000, 128, 8, 500, 4.0), (3000, 129, 8, 500, 4.0), (3000, 256, 16, 700, 4.0), (3000, 257, 5, 700, 4.0), (3000, 388, 4, 900, 4.0),
    (3000, 512, 8, 900, 4.0), (1200, 128, 24, 400, 4.0), (1200, 25, 47, 60, 4.0), (1200, 16, 48, 60, 4.0), (1200, 17, 49, 60, 4.0),
])
@pytest.mark.parametrize("center", [True, False])
def test_the_path_does_not_depend_on_how_the_scan_was_cut(T, K, C, length, level, center):
    w = runs(T + K + C, 3, T, K, C, length, level)
    flags = sb.SEMICRF_CENTER if center else 0
    ref = decode(w, flags)
    for extra in (sb.SEMICRF_SEQUENTIAL_SCAN, sb.SEMICRF_WARMUP(3 * K), sb.SEMICRF_WARMUP(5 * K + 7),
                  sb.SEMICRF_VITERBI_GLOBAL_TRACE, sb.SEMICRF_SEQUENTIAL_SCAN | sb.SEMICRF_VITERBI_GLOBAL_TRACE):
        got = decode(w, flags | extra)
        for name, a, b in zip(("labels", "starts", "nseg"), ref[1:], got[1:]):
            assert np.array_equal(a, b), (extra, name, int((a != b).sum()))
    check(w, center=center, label="runs longer than K")


def test_smallest_duration_and_label_among_equals():
    """All scores zero: every segmentation is as good as every other, so one-token segments of label 0."""
    w = synth.small_random(1, 2, 500, 9, 6, ragged=False)
    w.emis[:], w.trans[:], w.dur[:] = 0.0, 0.0, 0.0
    w.lengths[:] = [500, 333]
    score, labels, starts, nseg = decode(w, sb.SEMICRF_CENTER)
    for b, n in enumerate((500, 333)):
        assert score[b] == 0.0 and nseg[b] == n and (labels[b, :n] == 0).all() and (starts[b, :n] == 1).all()


def test_differences_above_rounding_decide():
    """Two durations whose biases differ by a float's last bits must not count as equal: 2 x (2 tokens) against 4 x (1 token)."""
    w = synth.small_random(2, 1, 400, 2, 1, ragged=False)
    w.emis[:], w.trans[:] = 0.0, 0.0
    for dur, n in (((1.0, np.nextafter(np.float32(2.0), np.float32(3.0))), 200), ((1.0, np.nextafter(np.float32(2.0), np.float32(1.0))), 400)):
        w.dur[:, 0] = dur
        assert decode(w, sb.SEMICRF_CENTER)[3][0] == n
