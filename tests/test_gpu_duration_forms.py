"""GPU parity of the duration, transition and emission statistics of long maximal durations (K >= 128), by the form that a call's
sizes lead to: tiles on the matrix cores, or vector multiply-adds where there are many workgroups with short intervals; and
inside the matrix-core launch vector multiply-adds for sequences with scaling blocks of fewer than sixteen positions.

Every case states its form, and the host's rule is worked out again from the sizes.  Tolerances as in test_gpu_duration_statistics:
1e-4 of the largest entry on the accumulated gradients and 1e-4 on what belongs to a position, against the oracle; 2e-6 of the largest entry
against the per-interval recurrence, 64-bit sums of up to 2500 terms rounded once to float.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def form(B, T, K, C, delta):
    labels = 4 if C <= 4 else 8                # a workgroup's; its eight waves share the durations, 128 at most to a wave
    parts = -(-K // (128 * (8 // labels)))
    workgroups = B * -(-T // delta) * -(-C // labels) * parts
    return "vector" if K < 192 and delta < 2 * K and workgroups > 512 else "matrix"


def check(B, T, K, C, delta, scale=1.0):  # scale: one, or one for each sequence
    w = synth.small_random(K + C, B, T, K, C, ragged=True, scale=1.0)
    w.emis *= np.broadcast_to(np.float32(scale), (B,))[:, None, None]
    w.lengths = np.maximum(w.lengths, 1)
    w.lengths[0] = T
    print(f"[case] B={B} T={T} K={K} C={C} delta={delta} scale={scale} {form(B, T, K, C, delta)}", flush=True)
    emis = w.emis.copy()
    for b in range(B):
        emis[b, int(w.lengths[b]):] = np.nan
    gl = np.linspace(0.5, 1.5, B)
    args = [torch.from_numpy(x).to(DEV) for x in (emis, w.lengths, w.trans, w.dur, gl.astype(np.float32))]
    ws = sb.alloc_workspace(B, T, K, C, delta, True)
    rows = sb.semicrf_fwd_bwd(*args, delta, workspace=ws)
    acc, _ = sb.semicrf_scan_report(ws, B, T, K, C, delta, True)
    recur = sb.semicrf_fwd_bwd(*args, delta, sb.SEMICRF_CENTER | sb.SEMICRF_MARGINALS_INTERVAL)
    torch.cuda.synchronize()
    assert acc.min().item() > 0                                      # the stored rows are used
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur, grad_logz=gl)
    for got, rec, name in zip(rows[1:], recur[1:], ("grad_emis", "grad_trans", "grad_dur", "pos_marg")):
        ref = getattr(r, name)
        top = 1.0 if name in ("grad_emis", "pos_marg") else max(1.0, np.abs(ref).max())
        got = got.double().cpu().numpy()
        rec = rec.double().cpu().numpy()
        print(f"       {name}: {np.abs(got - ref).max() / top:.1e}, recurrence {np.abs(got - rec).max() / top:.1e}", flush=True)
        assert np.abs(got - ref).max() <= 1e-4 * top, name
        assert np.abs(got - rec).max() <= 2e-6 * top, name


@pytest.mark.parametrize("B,T,K,C,delta", [
    (1, 333, 192, 5, 1),    # intervals of one position, two parts of the durations
    (1, 250, 140, 5, 1),
    (1, 333, 200, 3, 1),    # ... four labels a workgroup
    (2, 300, 256, 16, 15),  # two groups of labels and two parts, intervals that begin inside a tile
    (1, 500, 512, 8, 33),
])
def test_short_intervals_on_the_matrix_cores(B, T, K, C, delta):
    assert form(B, T, K, C, delta) == "matrix"
    check(B, T, K, C, delta)


@pytest.mark.parametrize("B,T,K,C,delta", [
    (32, 500, 128, 20, 80),   # groups of 32 positions, whole and not
    (48, 300, 160, 9, 100),
    (180, 260, 130, 3, 90),
    (300, 140, 191, 8, 70),
])
def test_vector_form_where_there_are_many_workgroups(B, T, K, C, delta):
    assert form(B, T, K, C, delta) == "vector"
    check(B, T, K, C, delta)


# Running sums of the emissions carried from chunk to chunk of an interval: 512 positions up to eight labels, 256 up to 16, 64 beyond;
# intervals that end inside a chunk, at its edge and just past it.
@pytest.mark.parametrize("T,K,C,delta", [
    (1100, 200, 13, 300),
    (1300, 200, 13, 520),
    (1000, 256, 16, 513),
    (2300, 192, 7, 600),
    (2300, 192, 7, 1100),
    (1500, 130, 4, 1025),
    (500, 128, 20, 200),
    (390, 128, 32, 129),
])
def test_intervals_of_several_chunks(T, K, C, delta):
    check(2, T, K, C, delta)


# Scaling blocks of fewer than sixteen positions (scores of N(0, 12^2)) in the matrix-core launch.
@pytest.mark.parametrize("B,T,K,C,delta", [
    (1, 2000, 512, 8, 1568),  # ranges of half of the durations: an interval's scales and all of them do not fit
    (1, 1700, 505, 6, 1600),  # ... which are not equal
    (1, 900, 512, 8, 392),    # one range, in the first of four parts
    (2, 400, 200, 13, 160),   # two groups of labels, the second not full
    (1, 600, 512, 3, 150),
])
def test_short_scaling_blocks_in_the_matrix_launch(B, T, K, C, delta):
    assert form(B, T, K, C, delta) == "matrix"
    check(B, T, K, C, delta, scale=12.0)


# Sequences of both kinds in one call: the first workgroups form other sequences' sums before their own.
@pytest.mark.parametrize("T,K,C,delta,scale", [
    (700, 300, 8, 100, (1.0, 12.0, 1.0, 12.0)),
    (600, 200, 13, 60, (12.0, 1.0, 1.0)),
    (500, 512, 4, 120, (1.0, 1.0, 12.0)),
])
def test_short_scaling_blocks_in_some_sequences(T, K, C, delta, scale):
    assert form(len(scale), T, K, C, delta) == "matrix"
    check(len(scale), T, K, C, delta, scale)
