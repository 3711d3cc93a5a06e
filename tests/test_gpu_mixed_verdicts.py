"""Sequences whose backward scan is accepted chunk by chunk while the forward scan is not: the interval kernels take them, from
windows that a short warm-up may have left incomplete.  Rare durations, whose expected counts come from exactly those entries."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth
from test_gpu_parity import assert_outputs_match_oracle

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("K,C,delta", [(100, 16, 104), (128, 32, 128), (64, 64, 64)])
def test_rare_durations_with_a_sequential_forward_scan(K, C, delta):
    """Two halves of the labels, alike in everything, between which a segment may change at a cost only and to one label only.  The
    first tokens pin the half; behind them nothing tells the halves apart (there is one long run of a label, or of its like).  A forward task that begins there with both halves
    equal is wrong however long it warms up; a backward task that does so is right."""
    pinned, T, half = 8 * C, 8 * C + 2200, C // 2
    w = synth.small_random(K + C, 1, T, K, C, ragged=False)
    w.emis[:, :pinned] = 0.0
    label = np.arange(pinned) // 8
    w.emis[:, np.arange(pinned), (label + half) % C] = 12.0  # every label as long: their means stay alike
    top = (pinned + 1500) // delta * delta
    w.emis[:, top - K: top + K, 1] += 6.0  # one long run across an interval's end
    w.emis[:, pinned:, half:] = w.emis[:, pinned:, :half]
    w.trans[:] = -1e4
    w.trans[:half, :half] = w.trans[half:, half:] = 0.0
    w.trans[np.arange(C), (np.arange(C) + half) % C] = -3.0
    w.dur[:, half:] = w.dur[:, :half]
    r = oracle.fwd_bwd(w.emis, w.lengths, w.trans, w.dur)
    ws = sb.alloc_workspace(w.B, T, K, C, delta, 1, "cuda:0").fill_(255)
    out = sb.semicrf_fwd_bwd(dev(w.emis), dev(w.lengths), dev(w.trans), dev(w.dur), None, delta, workspace=ws)
    acc = sb.semicrf_scan_report(ws, w.B, T, K, C, delta, 1)[0].cpu().numpy()
    out = [o.double().cpu().numpy() for o in out]
    some = r.grad_dur > 1e-30
    rel = np.abs(out[3] - r.grad_dur)[some] / r.grad_dur[some]
    print(f"[case] K={K} C={C} verified at {acc.tolist()}, relative error of grad_dur {rel.max():.1e} down to {r.grad_dur[some].min():.1e}", flush=True)
    assert (acc[:, 0] == 0).all() and (acc[:, 1] >= 1).all()
    assert_outputs_match_oracle(out, r)
    assert rel.max() <= 1e-6  # the rounding of the float; the scans agree to 2e-10 a boundary
