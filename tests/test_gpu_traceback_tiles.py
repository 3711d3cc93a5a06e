"""GPU tests of the Viterbi trace-back in tiles: paths whose tiles do not agree at first, and sequence lengths at the edges of
pieces and tiles.  Checked against the oracle's path scorer (test_gpu_viterbi.check) and, element by element, against the
trace-back by pointer doubling over all nodes, which has no tiles.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_viterbi import check, dev

pytestmark = pytest.mark.gpu


def decode(w, flags):
    out = sb.semicrf_viterbi(dev(w.emis), dev(w.lengths, np.int32), dev(w.trans), dev(w.dur), flags=flags)
    return [o.cpu().numpy() for o in out]


def both_routes(w, flags=sb.SEMICRF_CENTER):
    a, b = decode(w, flags), decode(w, flags | sb.SEMICRF_VITERBI_GLOBAL_TRACE)
    for name, x, y in zip(("score", "labels", "starts", "nseg"), a, b):
        assert np.array_equal(x, y), (name, np.argwhere(x != y)[:4])
    return a


@pytest.mark.parametrize("K,C", [(2, 2), (7, 3), (40, 3), (64, 24), (300, 8), (30, 64)])
def test_many_adjacent_tiles_are_traced_again(K, C):
    """Labels that may not follow each other: two labels, the worse of which leads for the first 60 % of the sequence.  Every
    tile there is first traced from the leading label's node and has to be traced again, from the root down, one by one."""
    B, T = 3, 4000
    w = synth.small_random(K, B, T, K, C, ragged=False)
    w.lengths[:] = [T, T - 1, T - 300]
    w.trans[:] = np.where(np.eye(C, dtype=bool), 0.0, -1.0e4)
    w.dur[:] = 0.0
    rng = np.random.default_rng(K)
    w.emis[:] = 0.01 * rng.standard_normal((B, T, C)) - 1.0
    w.emis[:, :int(0.6 * T), 0] += 1.0 + 0.2
    w.emis[:, :, C - 1] += 1.0
    w.emis[:, int(0.6 * T):, C - 1] += 0.9
    _, labels, _, _ = both_routes(w, flags=0)
    for b in range(B):
        L = int(w.lengths[b])
        assert np.all(labels[b, :L] == C - 1)
        lead = np.cumsum(w.emis[b].astype(np.float64), axis=0)[:L, 0] > np.cumsum(w.emis[b].astype(np.float64), axis=0)[:L, C - 1]
        assert lead[:2400].all()                   # at least four tiles of the largest size, one below the other
    check(w, center=False, label="labels that may not change")


@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 769])
@pytest.mark.parametrize("K,C", [(5, 3), (40, 24), (300, 8), (30, 64), (25, 47), (48, 33)])
def test_lengths_at_the_edges_of_pieces_and_tiles(T, K, C):
    """Pieces of 8, 4 (40 x 24) and 2 tokens (30 x 64), tiles of 32 of them, K longer than a tile; lengths
    that end one token into a tile or fill it."""
    w = synth.small_random(1000 * K + T, 3, T, K, C, ragged=False)
    w.lengths[:] = [T, max(1, T - 1), T // 2]
    both_routes(w)
    check(w, label="edges")
