"""GPU parity of the duration statistics of long maximal durations (K >= 128): the matrix-core form, whose tiles hold sixteen
positions by sixteen rows, and the form for scaling blocks shorter than a tile.

Sizes at the edges of that form: K at and next to multiples of 16 and of the shares of a wave, of a workgroup and of several
workgroups; labels below, at and beyond a workgroup's; intervals that begin inside a tile, are shorter than one, and are shorter than K;
sequences that end inside and at the edge of a tile.  Tolerances as in test_gpu_parity: 1e-4 of the largest
entry on the accumulated gradients, and against the per-interval recurrence (the same sums in another order) 2e-6 of it, 64-bit sums of
up to 2000 terms rounded once to float.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,T,K,C,delta,scale", [
    (1, 700, 128, 3, 0, 1.0),       # four labels a workgroup, two ranges of durations
    (2, 900, 257, 4, 0, 1.0),       # ... of five tiles of sixteen, in two parts
    (1, 1500, 512, 4, 0, 1.0),      # ... of eight
    (3, 500, 129, 8, 0, 1.0),       # one group of labels, two parts of the durations
    (1, 800, 192, 7, 104, 1.0),     # intervals that begin inside a tile of sixteen positions
    (2, 1100, 256, 8, 0, 1.0),
    (1, 1300, 300, 8, 0, 1.0),      # three parts of the durations
    (1, 2000, 512, 8, 0, 1.0),
    (2, 600, 128, 24, 0, 1.0),      # three groups of labels
    (1, 700, 200, 13, 0, 1.0),      # two, the second not full
    (1, 400, 160, 8, 8, 1.0),       # intervals shorter than a tile and than the durations
    (1, 333, 140, 5, 1, 1.0),       # ... of one position: 666 workgroups, so the vector form
    (2, 400, 128, 6, 0, 12.0),      # scaling blocks shorter than a tile
    (2, 300, 300, 8, 0, 30.0),
    (2, 260, 128, 20, 0, 12.0),
])
def test_duration_statistics_of_long_durations(B, T, K, C, delta, scale):
    w = synth.small_random(K + C, B, T, K, C, ragged=True, scale=scale)
    w.lengths[0] = T if delta else (T - T % 16)
    print(f"[case] B={B} T={T} K={K} C={C} delta={delta} scale={scale} lengths={w.lengths.tolist()}", flush=True)
    emis = w.emis.copy()
    for b in range(B):
        emis[b, int(w.lengths[b]):] = np.nan
    gl = np.linspace(0.5, 1.5, B)
    args = [torch.from_numpy(x).to(DEV) for x in (emis, w.lengths, w.trans, w.dur, gl.astype(np.float32))]
    ws = sb.alloc_workspace(B, T, K, C, delta, True)
    rows = sb.semicrf_fwd_bwd(*args, delta, workspace=ws)
    acc, _ = sb.semicrf_scan_report(ws, B, T, K, C, delta, True)
    again = sb.semicrf_fwd_bwd(*args, delta, workspace=ws)
    recur = sb.semicrf_fwd_bwd(*args, delta, sb.SEMICRF_CENTER | sb.SEMICRF_MARGINALS_INTERVAL)
    torch.cuda.synchronize()
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, grad_logz=gl)
    d = rows[3].double().cpu().numpy()
    top = max(1.0, np.abs(r.grad_dur).max())
    print(f"       verified at {acc.tolist()}, error {np.abs(d - r.grad_dur).max() / top:.1e}", flush=True)
    assert acc.min().item() > 0                                      # no pair went to the sequential scan
    assert np.abs(d - r.grad_dur).max() <= 1e-4 * top
    assert np.abs(rows[2].double().cpu().numpy() - r.grad_trans).max() <= 1e-4 * max(1.0, np.abs(r.grad_trans).max())
    assert np.abs(rows[4].double().cpu().numpy() - r.pos_marg).max() <= 1e-4
    assert (rows[3] - recur[3]).abs().max().item() <= 2e-6 * top
    assert all(torch.equal(x, y) for x, y in zip(rows, again))
